// z4c_tile.h -- device templates of the tile kernels (included by the
// per-variant translation units z4c_variants_*.hip).
#pragma once
// Tile kernels (one workgroup = one tile of TX*TY*TZ interior points of a
// MeshBlock, one point per thread).  The state fields are staged one at a
// time into LDS from a (TX+2R)(TY+2R)(TZ+2R) halo box, R = p/2 + 1 (the
// Kreiss-Oliger half width); while a field is being differentiated the next
// field's points are already in flight from HBM into registers.  Each
// field's derivatives are consumed at once in a fixed order (stage kernel:
// shift -> conformal metric -> Gamma-tilde -> lapse -> chi -> Khat, Theta ->
// At) so that the 66 first and 66 second derivatives of the Z4c right-hand
// side are never all live together, and each field's Runge-Kutta update is
// applied as soon as its right-hand side is complete.
//
// Stencils are centred, of order p = 4 or 6 (Sec. 4 uses 6), applied in
// centre-subtracted form (u_m - u_-m, u_m - u_0), mixed second derivatives
// as the first-derivative stencil applied along one axis to first
// differences along the other; Kreiss-Oliger dissipation of order p + 2 on
// every field (Sec. 4, sigma_KO).  The pointwise algebra is the standard
// Z4c system with constraint damping kappa1, kappa2 and the moving-puncture
// gauge (Sec. 2, Sec. 4), with the perfect-fluid ADM sources rho, S_i,
// S_ij (Sec. 2.1) as inputs.
//
// Arithmetic type R: double, or float with every stencil difference formed
// in double first (storage, Runge-Kutta combination and floors stay double).
#include <cmath>
#include <type_traits>
#include <utility>

#include "z4c_internal.h"

namespace z4c {
namespace tile {

constexpr double PI = 3.14159265358979323846;
constexpr int LDS_PER_CU = 163840;   // gfx950

// Symmetric 3x3 index: xx 0, xy 1, xz 2, yy 3, yz 4, zz 5.
__host__ __device__ constexpr int S(int i, int j)
{
    const int a = i < j ? i : j, b = i < j ? j : i;
    return a == 0 ? b : (a == 1 ? 2 + b : 5);
}
// Weight of a symmetric component in a full double contraction.
__host__ __device__ constexpr int SW(int a) { return (a == 1 || a == 2 || a == 4) ? 2 : 1; }
__host__ __device__ constexpr int SI(int a) { return a < 3 ? 0 : (a < 5 ? 1 : 2); }
__host__ __device__ constexpr int SJ(int a) { return a == 0 ? 0 : (a == 1 ? 1 : (a == 2 ? 2 : (a == 3 ? 1 : 2))); }

// LDS x pitch: the smallest value >= lx that is 8 mod 16 doubles, so that
// neighbouring rows of a wave's 8x8 footprint fall into disjoint banks.
constexpr int pad_pitch(int lx)
{
    int p = lx;
    while (p % 16 != 8)
        ++p;
    return p;
}

// ---------------------------------------------------------------------------
// 1-D stencils on LDS (centre pointer c, compile-time stride ST), unscaled
// ---------------------------------------------------------------------------
template <int P, typename R, int ST>
__device__ __forceinline__ R d1raw(const double *c)
{
    if constexpr (P == 4) {
        return R(8) * R(c[ST] - c[-ST]) - R(c[2 * ST] - c[-2 * ST]);
    } else {
        return R(45) * R(c[ST] - c[-ST]) - R(9) * R(c[2 * ST] - c[-2 * ST])
               + R(c[3 * ST] - c[-3 * ST]);
    }
}

template <int P, typename R, int ST>
__device__ __forceinline__ R d2raw(const double *c)
{
    const double c0 = c[0];
    if constexpr (P == 4) {
        return R(16) * R((c[ST] - c0) + (c[-ST] - c0))
               - R((c[2 * ST] - c0) + (c[-2 * ST] - c0));
    } else {
        return R(270) * R((c[ST] - c0) + (c[-ST] - c0))
               - R(27) * R((c[2 * ST] - c0) + (c[-2 * ST] - c0))
               + R(2) * R((c[3 * ST] - c0) + (c[-3 * ST] - c0));
    }
}

template <typename R>
struct Fac {
    R d1[3], d2[3], mix[3], ko[3];   // mix: xy, xz, yz
};

// Mixed second derivatives in two passes, x/y first (the constraint
// kernel's form; the stage kernel's z-first form follows): every
// thread first writes unscaled x- and y-first-derivative sums of the staged
// field over the tile extended by the stencil half width in the other
// directions (x sums: y and z extended; y sums: z extended); after a
// barrier, d_x d_y, d_x d_z and d_y d_z are first-derivative stencils on
// those sums (the tensor-product stencil).
template <int P, int TX, int TY, int TZ>
struct MixDims {
    static constexpr int Q = P / 2;
    static constexpr int DY = TY + 2 * Q, DZ = TZ + 2 * Q;
    static constexpr int NXS = TX * DY * DZ;   // x sums
    static constexpr int NYS = TX * TY * DZ;   // y sums
};

template <int P, typename R, int TX, int TY, int TZ, int PX, int PXY>
__device__ __forceinline__ void mix_prep(const double *L, R *dxb, R *dyb, int t)
{
    using M = MixDims<P, TX, TY, TZ>;
    constexpr int NT = TX * TY * TZ, RAD = P / 2 + 1, Q = M::Q;
#pragma unroll
    for (int q = 0; q < (M::NXS + NT - 1) / NT; ++q) {
        const int e = t + q * NT;
        if ((q + 1) * NT <= M::NXS || e < M::NXS) {
            const int ex = e % TX, r = e / TX, ey = r % M::DY, ez = r / M::DY;
            dxb[e] = d1raw<P, R, 1>(L + (ez - Q + RAD) * PXY + (ey - Q + RAD) * PX + (ex + RAD));
        }
    }
#pragma unroll
    for (int q = 0; q < (M::NYS + NT - 1) / NT; ++q) {
        const int e = t + q * NT;
        if ((q + 1) * NT <= M::NYS || e < M::NYS) {
            const int ex = e % TX, r = e / TX, ey = r % TY, ez = r / TY;
            dyb[e] = d1raw<P, R, PX>(L + (ez - Q + RAD) * PXY + (ey + RAD) * PX + (ex + RAD));
        }
    }
}

template <int P, typename R, int ST>
__device__ __forceinline__ R d1sum(const R *c)
{
    if constexpr (P == 4)
        return R(8) * (c[ST] - c[-ST]) - (c[2 * ST] - c[-2 * ST]);
    else
        return R(45) * (c[ST] - c[-ST]) - R(9) * (c[2 * ST] - c[-2 * ST]) + (c[3 * ST] - c[-3 * ST]);
}

// Two-pass mixed derivatives of the stage kernel, z-pass first: zs = D_z u
// over the tile extended by Q in x and y, ys = D_y u over the tile extended
// by Q in x (unscaled sums); then xz = D_x(zs), yz = D_y(zs), xy = D_x(ys).
// A z plane of NR rows of at most 16 sums: even rows 16 apart from the
// plane's start, odd rows 16 apart from an offset of 8 mod 16, so that for
// double sums any run of two to four consecutive rows, each read at 8
// consecutive x (the 8x8 footprint of a wave), falls in distinct LDS banks
// (rows r..r+3 start at 0, 8, 16, 24 mod 32 doubles in some order);
// consecutive rows at a pitch of 14 or 12 sums would share banks.
template <int NR>
struct SumRows {
    static constexpr int OFF = 16 * ((NR + 1) / 2) + 8;
    static constexpr int PLANE = OFF + 16 * (NR / 2);
    __host__ __device__ static constexpr int row(int r) { return (r & 1) * OFF + (r >> 1) * 16; }
};

template <int P, int TX, int TY, int TZ>
struct MixDimsZ {
    static constexpr int Q = P / 2;
    static constexpr int EX = TX + 2 * Q, EY = TY + 2 * Q;
    static_assert(EX <= 16, "a row of sums spans at most 16 x");
    using ZR = SumRows<EY>;                          // z sums: EY rows per plane
    using YR = SumRows<TY>;                          // y sums: TY rows per plane
    static constexpr int NZS = ZR::PLANE * TZ;       // storage, in sums
    static constexpr int NYS = YR::PLANE * TZ;
};

// First derivative along y of the z sums at row r of a plane, from pe = the
// sum at row r and po = the same x at row r + 1 (rows r + k: pe + 8k for even
// k, po + 8(k - 1) for odd k); the terms as in d1sum.
template <int P, typename R>
__device__ __forceinline__ R d1sum_rows(const R *pe, const R *po)
{
    if constexpr (P == 4)
        return R(8) * (po[0] - po[-16]) - (pe[16] - pe[-16]);
    else
        return R(45) * (po[0] - po[-16]) - R(9) * (pe[16] - pe[-16]) + (po[16] - po[-32]);
}

// Unfused helpers used by the constraint kernel.
template <int P, typename R, int PX, int PXY>
__device__ __forceinline__ void first(const double *c, const Fac<R> &F, R d[3])
{
    d[0] = d1raw<P, R, 1>(c) * F.d1[0];
    d[1] = d1raw<P, R, PX>(c) * F.d1[1];
    d[2] = d1raw<P, R, PXY>(c) * F.d1[2];
}

// Second derivatives, the mixed ones from the two-pass sums of mix_prep
// (dxb, dyb).
template <int P, typename R, int PX, int PXY, int TX, int TY, int TZ>
__device__ __forceinline__ void second_sums(const double *c, const Fac<R> &F, R dd[6],
                                            const R *dxb, const R *dyb, int tx, int ty, int tz)
{
    using M = MixDims<P, TX, TY, TZ>;
    dd[0] = d2raw<P, R, 1>(c) * F.d2[0];
    dd[3] = d2raw<P, R, PX>(c) * F.d2[1];
    dd[5] = d2raw<P, R, PXY>(c) * F.d2[2];
    const R *px = dxb + ((tz + M::Q) * M::DY + (ty + M::Q)) * TX + tx;
    const R *py = dyb + ((tz + M::Q) * TY + ty) * TX + tx;
    dd[1] = d1sum<P, R, TX>(px) * F.mix[0];
    dd[2] = d1sum<P, R, TX * M::DY>(px) * F.mix[1];
    dd[4] = d1sum<P, R, TX * TY>(py) * F.mix[2];
}

template <typename R>
__device__ __forceinline__ R symtrace(const R gi[6], const R t[6])
{
    return gi[0] * t[0] + gi[3] * t[3] + gi[5] * t[5]
           + R(2) * (gi[1] * t[1] + gi[2] * t[2] + gi[4] * t[4]);
}

// Logical workgroup index: consecutive logical indices on the same XCD
// (the dispatcher places workgroup w on XCD w % 8).
__device__ __forceinline__ int xcd_logical(int w, int G)
{
    const int q = G >> 3, r = G & 7;
    const int x = w & 7, k = w >> 3;
    return x * q + (x < r ? x : r) + k;
}

// Tile of this workgroup: one workgroup per tile, workgroup w taking the tile
// of logical index xcd_logical(w), so that consecutive tiles (neighbours in
// one block, which share halo points) run on one XCD and meet in its L2.
__device__ __forceinline__ int my_tile() { return xcd_logical(blockIdx.x, gridDim.x); }

// Algebraic enforcement after a stage (double): det(gt) = 1, tr(At) = 0, floors.
__device__ __forceinline__ void enforce(double v[NFIELD], double chi_floor, double alpha_floor)
{
    double g[6];
#pragma unroll
    for (int a = 0; a < 6; ++a)
        g[a] = v[GXX + a];
    double det = g[0] * (g[3] * g[5] - g[4] * g[4]) - g[1] * (g[1] * g[5] - g[4] * g[2])
               + g[2] * (g[1] * g[4] - g[3] * g[2]);
    const double f = 1.0 / cbrt(det);
#pragma unroll
    for (int a = 0; a < 6; ++a)
        g[a] *= f;
    det = g[0] * (g[3] * g[5] - g[4] * g[4]) - g[1] * (g[1] * g[5] - g[4] * g[2])
        + g[2] * (g[1] * g[4] - g[3] * g[2]);
    const double id = 1.0 / det;
    double gi[6];
    gi[0] = (g[3] * g[5] - g[4] * g[4]) * id;
    gi[1] = (g[2] * g[4] - g[1] * g[5]) * id;
    gi[2] = (g[1] * g[4] - g[2] * g[3]) * id;
    gi[3] = (g[0] * g[5] - g[2] * g[2]) * id;
    gi[4] = (g[2] * g[1] - g[0] * g[4]) * id;
    gi[5] = (g[0] * g[3] - g[1] * g[1]) * id;
    double A[6];
#pragma unroll
    for (int a = 0; a < 6; ++a)
        A[a] = v[AXX + a];
    const double tr = gi[0] * A[0] + gi[3] * A[3] + gi[5] * A[5]
                    + 2.0 * (gi[1] * A[1] + gi[2] * A[2] + gi[4] * A[4]);
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        v[GXX + a] = g[a];
        v[AXX + a] = A[a] - g[a] * tr * (1.0 / 3.0);
    }
    v[CHI] = v[CHI] > chi_floor ? v[CHI] : chi_floor;
    v[ALPHA] = v[ALPHA] > alpha_floor ? v[ALPHA] : alpha_floor;
}

// ---------------------------------------------------------------------------
// The tile kernel
// ---------------------------------------------------------------------------
template <typename Fn, int... Is>
__device__ __forceinline__ void sfor_impl(Fn &&f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
// Compile-time loop: f(std::integral_constant<int, i>) for i = 0 .. N-1.
template <int N, typename Fn>
__device__ __forceinline__ void sfor(Fn &&f)
{
    sfor_impl(f, std::make_integer_sequence<int, N>{});
}

// Field staged after field f (-1: none).  Constraints: gt, Gt, chi, Khat,
// Theta, At.  Right-hand side / stage: beta, gt, Gt, alpha, chi, Khat,
// Theta, At.
template <int MODE>
__host__ __device__ constexpr int next_field(int f)
{
    if (MODE != MODE_CONS) {
        if (f == BETAX || f == BETAY)
            return f + 1;
        if (f == BETAZ)
            return GXX;
    }
    if (f >= GXX && f < GZZ)
        return f + 1;
    if (f == GZZ)
        return GAMX;
    if (f == GAMX || f == GAMY)
        return f + 1;
    if (f == GAMZ)
        return MODE == MODE_CONS ? CHI : ALPHA;
    if (f == ALPHA)
        return CHI;
    if (f == CHI)
        return KHAT;
    if (f == KHAT)
        return THETA;
    if (f == THETA)
        return AXX;
    if (f >= AXX && f < AZZ)
        return f + 1;
    return -1;
}

// Element at byte offset `boff` from a (wave-uniform) base in global memory: a
// 32-bit offset added to a scalar base, the addressing form that needs no
// 64-bit per-lane address.
typedef __attribute__((address_space(1))) double gdouble;
__device__ __forceinline__ const gdouble &at(const double *b, unsigned boff)
{
    return *(const gdouble *)((const __attribute__((address_space(1))) char *)b + boff);
}
__device__ __forceinline__ gdouble &at(double *b, unsigned boff)
{
    return *(gdouble *)((__attribute__((address_space(1))) char *)b + boff);
}

// Entry n of a table that no kernel writes (tiles, blocks, stencil factors),
// read through the constant address space: a uniform index gives scalar
// loads, also where the kernel has stored to global memory before.
template <typename T>
__device__ __forceinline__ T read_words(const __attribute__((address_space(4))) unsigned *c)
{
    static_assert(sizeof(T) % 4 == 0, "whole words");
    struct Words {
        unsigned w[sizeof(T) / 4];
    } x;
#pragma unroll
    for (unsigned q = 0; q < sizeof(T) / 4; ++q)
        x.w[q] = c[q];
    return __builtin_bit_cast(T, x);
}
template <typename T>
__device__ __forceinline__ T table_entry(const T *p, long long n)
{
    return read_words<T>(
        (const __attribute__((address_space(4))) unsigned *)(unsigned long long)(p + n));
}
// Halo-tile staging of one field at a time: registers <- HBM (prefetch of
// the next field), LDS <- registers (between two barriers).  Each halo
// element has a 32-bit element offset found once per tile: from the block's
// own base of field 0 for its own points and stored ghosts, the periodic
// image and the same point of `frozen`; from the state array base for
// another block's point under the neighbour rule (the plan refuses that rule
// unless such offsets stay below 2^32).  Blocks of the first kind may lie
// anywhere in the state array.
template <int NLD>
struct Stager {
    int ldo[NLD];
    unsigned src[NLD];
    unsigned valid, frz, far;   // bit q: element q is loaded / from `frozen` / from another block
    double pf[NLD];
    const double *own, *own_frozen, *all;   // u + offset, frozen + offset, u
    long long fs;

    __device__ __forceinline__ void prefetch(int f)
    {
        const long long e = (long long)f * fs;   // uniform
#pragma unroll
        for (int q = 0; q < NLD; ++q)
            pf[q] = (valid >> q) & 1u
                        ? ((far >> q) & 1u ? all + e : (frz >> q) & 1u ? own_frozen + e : own + e)[src[q]]
                        : 0.0;
    }
    __device__ __forceinline__ void store(double *lds)
    {
#pragma unroll
        for (int q = 0; q < NLD; ++q)
            if (ldo[q] >= 0)
                lds[ldo[q]] = pf[q];
    }
};

template <int NLD, int NT, int RAD, int LX, int LY, int LZ, int PX, int PXY>
__device__ __forceinline__ void setup_stager(Stager<NLD> &st, const StageArgs &a, const Tile &T,
                                             const z4c_block &B, int t)
{
    constexpr int LVOL = LX * LY * LZ;
    const int ng = B.ng;
    const int sy = B.nx + 2 * ng;
    const int sz = sy * (B.ny + 2 * ng);
    st.own = a.u + B.offset;
    st.own_frozen = a.frozen ? a.frozen + B.offset : nullptr;
    st.all = a.u;
    st.fs = B.field_stride;
    st.valid = 0u;
    st.frz = 0u;
    st.far = 0u;
#pragma unroll
    for (int q = 0; q < NLD; ++q) {
        const int e = t + q * NT;
        st.ldo[q] = -1;
        st.src[q] = 0u;
        if (e < LVOL) {
            const int lx = e % LX, r1 = e / LX, ly = r1 % LY, lz = r1 / LY;
            const int gi = T.i0 - RAD + lx, gj = T.j0 - RAD + ly, gk = T.k0 - RAD + lz;
            st.ldo[q] = lz * PXY + ly * PX + lx;
            if (gi >= -ng && gi < B.nx + ng && gj >= -ng && gj < B.ny + ng && gk >= -ng
                && gk < B.nz + ng) {
                const int ox = gi < 0 ? -1 : (gi >= B.nx ? 1 : 0);
                const int oy = gj < 0 ? -1 : (gj >= B.ny ? 1 : 0);
                const int oz = gk < 0 ? -1 : (gk >= B.nz ? 1 : 0);
                unsigned idx = (unsigned)((gk + ng) * sz + (gj + ng) * sy + (gi + ng));
                if ((ox | oy | oz) != 0 && a.halo != Z4C_GHOST_NONE) {
                    int sb = -1;
                    if (a.halo == Z4C_GHOST_PERIODIC)
                        sb = T.block;
                    else if (a.halo == Z4C_GHOST_NEIGHBOUR)
                        sb = a.nbr[T.block * 27 + (oz + 1) * 9 + (oy + 1) * 3 + (ox + 1)];
                    if (sb >= 0) {
                        // same nx, ny, nz, ng and field stride as this block
                        const int si = gi - ox * B.nx, sj = gj - oy * B.ny, sk = gk - oz * B.nz;
                        idx = (unsigned)((sk + ng) * sz + (sj + ng) * sy + (si + ng));
                        if (sb != T.block) {
                            idx += (unsigned)a.blocks[sb].offset;
                            st.far |= 1u << q;
                        }
                    } else if (a.frozen) {
                        st.frz |= 1u << q;
                    }   // else: the stored ghost, which a refresh leaves as it is
                }
                st.src[q] = idx;
                st.valid |= 1u << q;
            }
        }
    }
}

template <int P, int TX, int TY, int TZ, typename R>
__global__ void __launch_bounds__(TX *TY *TZ) cons_kernel(const StageArgs a)
{
    constexpr int RAD = P / 2 + 1;
    constexpr int NT = TX * TY * TZ;
    constexpr int LX = TX + 2 * RAD, LY = TY + 2 * RAD, LZ = TZ + 2 * RAD;
    constexpr int PX = pad_pitch(LX);
    constexpr int PXY = PX * LY;
    constexpr int LVOL = LX * LY * LZ;
    constexpr int NLD = (LVOL + NT - 1) / NT;
    __shared__ double lds[PXY * LZ];
    __shared__ double red[(NT / 64) * 16];
    // mixed second derivatives of chi and gt in two passes (as the stage
    // kernel): x and y first-derivative sums here
    using MD = MixDims<P, TX, TY, TZ>;
    __shared__ R dxb[MD::NXS];
    __shared__ R dyb[MD::NYS];

    const int t = threadIdx.x;
    const int tx = t % TX, ty = (t / TX) % TY, tz = t / (TX * TY);
    const double *lc = lds + (tz + RAD) * PXY + (ty + RAD) * PX + (tx + RAD);

    {
        const int tile = my_tile();
        const Tile T = a.tiles[tile];
        const z4c_block B = a.blocks[T.block];
        const int ng = B.ng;
        const int sy = B.nx + 2 * ng;
        const int sz = sy * (B.ny + 2 * ng);
        const int i = T.i0 + tx, j = T.j0 + ty, k = T.k0 + tz;
        const bool active = i < B.nx && j < B.ny && k < B.nz;
        const int pt = (k + ng) * sz + (j + ng) * sy + (i + ng);
        const double *ub = a.u + B.offset;
        const long long fs = B.field_stride;

        Stager<NLD> st;
        setup_stager<NLD, NT, RAD, LX, LY, LZ, PX, PXY>(st, a, T, B, t);
        auto stage = [&](auto FC) __attribute__((always_inline)) {
            constexpr int FF = decltype(FC)::value;
            constexpr int NX = next_field<MODE_CONS>(FF);
            __syncthreads();
            st.store(lds);
            if constexpr (NX >= 0)
                st.prefetch(NX);
            __syncthreads();
            if constexpr (FF == CHI || (FF >= GXX && FF <= GZZ)) {
                mix_prep<P, R, TX, TY, TZ, PX, PXY>(lds, dxb, dyb, t);
                __syncthreads();
            }
        };

        st.prefetch(GXX);

        const Fac<R> F = table_entry((const Fac<R> *)a.fac64, T.block);
        // Conformal metric, its inverse; conformal factor.
        R g[6];
        sfor<6>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; { g[q] = active ? R(ub[(GXX + q) * fs + pt]) : ((q == 0 || q == 3 || q == 5) ? R(1) : R(0)); } });
        R gi[6];
        {
            const R det = g[0] * (g[3] * g[5] - g[4] * g[4]) - g[1] * (g[1] * g[5] - g[4] * g[2])
                        + g[2] * (g[1] * g[4] - g[3] * g[2]);
            const R id = R(1) / det;
            gi[0] = (g[3] * g[5] - g[4] * g[4]) * id;
            gi[1] = (g[2] * g[4] - g[1] * g[5]) * id;
            gi[2] = (g[1] * g[4] - g[2] * g[3]) * id;
            gi[3] = (g[0] * g[5] - g[2] * g[2]) * id;
            gi[4] = (g[2] * g[1] - g[0] * g[4]) * id;
            gi[5] = (g[0] * g[3] - g[1] * g[1]) * id;
        }
        const R chi = active ? R(ub[CHI * fs + pt]) : R(1);
        const R chis = chi > R(a.chi_floor) ? chi : R(a.chi_floor);
        const R ichi2 = R(0.5) / chis;          // 1 / (2 chi)
        R cons[NCONS];
        sfor<NCONS>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; { cons[q] = R(0); } });

        // ---- conformal metric: d gt, d d gt -> Rt_ij (second-derivative part)
        R dg[3][6];
        R Rij[6];
        sfor<6>([&](auto Q) __attribute__((always_inline)) {
            constexpr int q = decltype(Q)::value;
            stage(std::integral_constant<int, GXX + q>{});
            if (active) {
                R d[3], dd[6];
                first<P, R, PX, PXY>(lc, F, d);
                second_sums<P, R, PX, PXY, TX, TY, TZ>(lc, F, dd, dxb, dyb, tx, ty, tz);
                sfor<3>([&](auto kk_c) __attribute__((always_inline)) { constexpr int kk = decltype(kk_c)::value; { dg[kk][q] = d[kk]; } });
                Rij[q] = R(-0.5) * symtrace(gi, dd);
            }
        });

        // Christoffel symbols: Gl[k][ij] = Gt_{k ij}, Gu[k][ij] = Gt^k_{ij}, Gd^i.
        R Gu[3][6], Gd[3];
        if (active) {
            R Gl[3][6];
            sfor<3>([&](auto kk_c) __attribute__((always_inline)) { constexpr int kk = decltype(kk_c)::value; {                 sfor<6>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; {
                    const int ii = SI(q), jj = SJ(q);
                    Gl[kk][q] = R(0.5) * (dg[ii][S(jj, kk)] + dg[jj][S(ii, kk)] - dg[kk][q]);
                } }); } });
            sfor<3>([&](auto kk_c) __attribute__((always_inline)) { constexpr int kk = decltype(kk_c)::value; {                 sfor<6>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; { Gu[kk][q] = gi[S(kk, 0)] * Gl[0][q] + gi[S(kk, 1)] * Gl[1][q]
                              + gi[S(kk, 2)] * Gl[2][q]; } }); } });
            sfor<3>([&](auto ii_c) __attribute__((always_inline)) { constexpr int ii = decltype(ii_c)::value; { Gd[ii] = symtrace(gi, Gu[ii]); } });
            // Rt_ij += 1/2 Gd^k (Gt_{ijk} + Gt_{jik})
            //        + sum_kl (Gu^k_{li} T_{jk}^l + Gu^k_{lj} T_{ik}^l + Gu^k_{il} T_{kj}^l),
            // T_{ab}^c = gt^{cm} Gt_{a bm}
            sfor<6>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; {
                const int ii = SI(q), jj = SJ(q);
                R s = R(0);
                sfor<3>([&](auto kk_c) __attribute__((always_inline)) { constexpr int kk = decltype(kk_c)::value; { s += R(0.5) * Gd[kk] * (Gl[ii][S(jj, kk)] + Gl[jj][S(ii, kk)]); } });
                Rij[q] += s;
            } });
            sfor<3>([&](auto p0_c) __attribute__((always_inline)) { constexpr int p0 = decltype(p0_c)::value; {                 sfor<3>([&](auto p1_c) __attribute__((always_inline)) { constexpr int p1 = decltype(p1_c)::value; {
                    R Tc[3];
                    sfor<3>([&](auto p2_c) __attribute__((always_inline)) { constexpr int p2 = decltype(p2_c)::value; { Tc[p2] = gi[S(p2, 0)] * Gl[p0][S(p1, 0)] + gi[S(p2, 1)] * Gl[p0][S(p1, 1)]
                               + gi[S(p2, 2)] * Gl[p0][S(p1, 2)]; } });
                    // T_{p0 p1}^{l}: contributes as T_{jk}^l (j=p0, k=p1),
                    // T_{ik}^l (i=p0, k=p1) and T_{kj}^l (k=p0, j=p1)
                    sfor<6>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; {
                        const int ii = SI(q), jj = SJ(q);
                        R s = R(0);
                        sfor<3>([&](auto l_c) __attribute__((always_inline)) { constexpr int l = decltype(l_c)::value; {
                            if (jj == p0)
                                s += Gu[p1][S(l, ii)] * Tc[l];
                            if (ii == p0)
                                s += Gu[p1][S(l, jj)] * Tc[l];
                            if (jj == p1)
                                s += Gu[p0][S(ii, l)] * Tc[l];
                        } });
                        Rij[q] += s;
                    } });
                } }); } });
        }

        // ---- Gamma-tilde: d_j Gt^k -> Rt_ij; damping; Z^i
        sfor<3>([&](auto KK) __attribute__((always_inline)) {
            constexpr int kk = decltype(KK)::value;
            stage(std::integral_constant<int, GAMX + kk>{});
            if (active) {
                R d[3];
                first<P, R, PX, PXY>(lc, F, d);
                sfor<6>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; {
                    const int ii = SI(q), jj = SJ(q);
                    Rij[q] += R(0.5) * (g[S(kk, ii)] * d[jj] + g[S(kk, jj)] * d[ii]);
                } });
                const R Gam = R(lc[0]);
                cons[C_ZX + kk] = R(0.5) * (Gam - Gd[kk]);
            }
        });

        // ---- chi: R^chi_ij
        R dchi[3];
        stage(std::integral_constant<int, CHI>{});
        if (active) {
            R dd[6];
            first<P, R, PX, PXY>(lc, F, dchi);
            second_sums<P, R, PX, PXY, TX, TY, TZ>(lc, F, dd, dxb, dyb, tx, ty, tz);
            R DD[6];
            sfor<6>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; { DD[q] = dd[q] - (Gu[0][q] * dchi[0] + Gu[1][q] * dchi[1] + Gu[2][q] * dchi[2]); } });
            const R trDD = symtrace(gi, DD);
            R dc2[6];
            sfor<6>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; { dc2[q] = dchi[SI(q)] * dchi[SJ(q)]; } });
            const R dchi2 = symtrace(gi, dc2);
            const R i4c2 = ichi2 * ichi2;   // 1 / (4 chi^2)
            sfor<6>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; { Rij[q] += (DD[q] + g[q] * trDD) * ichi2 - (dc2[q] + R(3) * g[q] * dchi2) * i4c2; } });
        }

        // ---- Khat, Theta (their Gamma-tilde source terms)
        R KT[2];
        sfor<2>([&](auto Q) __attribute__((always_inline)) {
            constexpr int q = decltype(Q)::value;
            stage(std::integral_constant<int, q == 0 ? KHAT : THETA>{});
            if (active) {
                R d[3];
                first<P, R, PX, PXY>(lc, F, d);
                KT[q] = R(lc[0]);
                const R c = q == 0 ? R(-2.0 / 3.0) : R(-4.0 / 3.0);
                sfor<3>([&](auto ii_c) __attribute__((always_inline)) { constexpr int ii = decltype(ii_c)::value; { cons[C_MX + ii] += c * d[ii]; } });
            }
        });

        // ---- pointwise algebra
        R A[6];
        if (active) {
            const R Khat = KT[0], Theta = KT[1];
            sfor<6>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; { A[q] = R(ub[(AXX + q) * fs + pt]); } });
            R rho = R(0), Si[3] = {R(0), R(0), R(0)}, Sij[6] = {R(0), R(0), R(0), R(0), R(0), R(0)};
            if (a.matter) {
                const double *mb = a.matter + B.moffset;
                rho = R(mb[pt]);
                sfor<3>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; { Si[q] = R(mb[(1 + q) * fs + pt]); } });
                sfor<6>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; { Sij[q] = R(mb[(4 + q) * fs + pt]); } });
            }
            // At^i_j and At^{ij}
            R Amix[3][3];
            sfor<3>([&](auto ii_c) __attribute__((always_inline)) { constexpr int ii = decltype(ii_c)::value; {                 sfor<3>([&](auto jj_c) __attribute__((always_inline)) { constexpr int jj = decltype(jj_c)::value; { Amix[ii][jj] = gi[S(ii, 0)] * A[S(0, jj)] + gi[S(ii, 1)] * A[S(1, jj)]
                                 + gi[S(ii, 2)] * A[S(2, jj)]; } }); } });
            R Aup[6];
            sfor<6>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; {
                const int ii = SI(q), jj = SJ(q);
                Aup[q] = Amix[ii][0] * gi[S(0, jj)] + Amix[ii][1] * gi[S(1, jj)]
                       + Amix[ii][2] * gi[S(2, jj)];
            } });
            R AA = R(0);
            sfor<6>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; { AA += R(SW(q)) * A[q] * Aup[q]; } });
            const R K = Khat + R(2) * Theta;
            const R Rs = chi * symtrace(gi, Rij);
            const R pi = R(PI);
            cons[C_H] = Rs + R(2.0 / 3.0) * K * K - AA - R(16) * pi * rho;
            cons[C_THETA] = Theta;
            sfor<3>([&](auto ii_c) __attribute__((always_inline)) { constexpr int ii = decltype(ii_c)::value; {
                R s = R(0);
                sfor<3>([&](auto jj_c) __attribute__((always_inline)) { constexpr int jj = decltype(jj_c)::value; {                         sfor<3>([&](auto kk_c) __attribute__((always_inline)) { constexpr int kk = decltype(kk_c)::value; {
                        R c2 = R(0);
                        sfor<3>([&](auto l_c) __attribute__((always_inline)) { constexpr int l = decltype(l_c)::value; { c2 += Gu[l][S(jj, kk)] * A[S(l, ii)] + Gu[l][S(jj, ii)] * A[S(kk, l)]; } });
                        s += gi[S(jj, kk)] * c2;
                    } }); } });
                const R Ac = Amix[0][ii] * dchi[0] + Amix[1][ii] * dchi[1]
                           + Amix[2][ii] * dchi[2];
                cons[C_MX + ii] += -s - R(1.5) / chis * Ac - R(8) * pi * Si[ii];
            } });
        }

        // ---- At_ij
        sfor<6>([&](auto Q) __attribute__((always_inline)) {
            constexpr int q = decltype(Q)::value;
            stage(std::integral_constant<int, AXX + q>{});
            if (active) {
                R d[3];
                first<P, R, PX, PXY>(lc, F, d);
                constexpr int ii = SI(q), jj = SJ(q);
                cons[C_MX + ii] += gi[S(jj, 0)] * d[0] + gi[S(jj, 1)] * d[1] + gi[S(jj, 2)] * d[2];
                if constexpr (ii != jj)
                    cons[C_MX + jj] += gi[S(ii, 0)] * d[0] + gi[S(ii, 1)] * d[1]
                                     + gi[S(ii, 2)] * d[2];
            }
        });

        // ---- output
        if (active && a.out) {
            double *cb = a.out + B.coffset;
            sfor<NCONS>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; { cb[q * fs + pt] = double(cons[q]); } });
        }
        // Per-tile sums of |c| and c^2 in a fixed order: wave reduction,
        // then the waves in order.
        double v[16];
        sfor<NCONS>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; {
            const double c = active ? double(cons[q]) : 0.0;
            v[2 * q] = fabs(c);
            v[2 * q + 1] = c * c;
        } });
        sfor<16>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1)
                v[q] += __shfl_xor(v[q], off, 64);
        } });
        const int wave = t >> 6, lane = t & 63;
        __syncthreads();
        if (lane == 0)
            sfor<16>([&](auto q_c) __attribute__((always_inline)) { constexpr int q = decltype(q_c)::value; { red[wave * 16 + q] = v[q]; } });
        __syncthreads();
        if (t < 16) {
            double s = 0.0;
            for (int w = 0; w < NT / 64; ++w)
                s += red[w * 16 + t];
            a.partial[tile * 16LL + t] = s;
        }
    }
}

}  // namespace tile

template <int P>
hipError_t launch_cons(const StageArgs &a, hipStream_t s)
{
    tile::cons_kernel<P, TILE_X, TILE_Y, TILE_Z, double>
        <<<a.ntiles, dim3(TILE_X * TILE_Y * TILE_Z), 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace z4c
