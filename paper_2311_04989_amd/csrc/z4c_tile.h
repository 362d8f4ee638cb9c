// z4c_tile.h -- device templates of the tile kernels (included by the
// per-variant translation units z4c_variants_*.hip).
#pragma once
// Tile kernels (one workgroup = one tile of TX*TY*TZ interior points of a
// MeshBlock, one point per thread).  The state fields are staged one at a
// time from a (TX+2R)(TY+2R)(TZ+2R) halo box, R = p/2 + 1 (the Kreiss-Oliger
// half width), into registers, a z-column per thread, and what the stencils of
// others read of it into LDS; while a field is being differentiated the next
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
constexpr int LDS_GRANULE = 1280;    // a workgroup's LDS is allocated in these

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

template <typename R>
struct Fac {
    R d1[3], d2[3], mix[3], ko[3];   // mix: xy, xz, yz
};

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
// Six sums are read per derivative where the tensor product of differences reads
// 36 values, at one rounding of the first derivative per point: off-diagonal
// right-hand sides of At on the 64^3 star have an rms error of 2.7e-15 of their
// size, by the tensor product 0.9e-15.
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

template <typename R>
__device__ __forceinline__ R symtrace(const R gi[6], const R t[6])
{
    return gi[0] * t[0] + gi[3] * t[3] + gi[5] * t[5]
           + R(2) * (gi[1] * t[1] + gi[2] * t[2] + gi[4] * t[4]);
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

// Field staged after field f (-1: none).  Constraints: chi, gt, Gt, Khat,
// Theta, At.  Right-hand side / stage: beta, gt, Gt, lapse, chi, Khat,
// Theta, At.
template <int MODE>
__host__ __device__ constexpr int next_field(int f)
{
    constexpr bool CONS = MODE == MODE_CONS;
    switch (f) {
    case BETAZ: return GXX;
    case GZZ: return GAMX;
    case GAMZ: return CONS ? KHAT : ALPHA;
    case ALPHA: return CHI;
    case CHI: return CONS ? GXX : KHAT;
    case KHAT: return THETA;
    case THETA: return AXX;
    case AZZ: return -1;
    default: return f + 1;   // components of one tensor
    }
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
// Staging by z-columns.  The halo box of a tile is LX x LY columns of LZ
// points; thread t holds the whole column (t mod LX, t / LX) of a field in
// registers.  What the stencils read of it goes to LDS: the x and y stencils
// need the TZ interior planes (PLN doubles each, rows PX apart), the z
// stencils only the TX x TY interior columns (NZC doubles, planes TX * TY
// apart), and the z sums of the mixed derivatives are formed from the
// registers.  That is 18 KB per field and tile instead of the whole box's
// 37 KB, and a field without second derivatives loads 1,280 points instead
// of 3,072.  With the sums and 25 values per thread parked in LDS, a
// workgroup takes half a CU's LDS and its lanes half a SIMD's registers: two
// workgroups per CU, whose barriers and memory waits cover one another.  That is
// without scratch but for order 6 in double: the monitor form spills 16 registers
// (22 with neighbour or frozen halos), the lopsided one 25 to 41, the plain one
// none (2).
template <int P, int TX, int TY, int TZ>
struct ColDims {
    static constexpr int RAD = P / 2 + 1, Q = P / 2, NT = TX * TY * TZ;
    static constexpr int LX = TX + 2 * RAD, LY = TY + 2 * RAD, LZ = TZ + 2 * RAD;
    static constexpr int PX = pad_pitch(LX), PLN = PX * LY;
    static constexpr int NPL = PLN * TZ, NZC = TX * TY * LZ;
    static_assert(LX * LY <= NT, "one column per thread");
    static_assert(TZ >= RAD, "at most the first tile of a block reaches below it");
};

// Fields with second derivatives.
__host__ __device__ constexpr bool mixed_field(int f)
{
    return f == CHI || f == ALPHA || (f >= GXX && f <= GZZ) || (f >= BETAX && f <= BETAZ);
}

// The column of one thread and where its points come from.  The refresh rule
// acts per direction, so the source of a point is the column's (x, y) part,
// fixed per thread, plus the plane's z part, the same for all threads: a
// byte offset per plane in scalar registers.
// GEN (frozen and neighbour rules): the array and block that the (x, y) part
// refers to depend on whether the plane lies below, in or above the block,
// so a thread keeps one pointer for each (`below`, `in`, `above`).
// KO: with the outermost points, which only the dissipation reads.
template <int P, int TX, int TY, int TZ, bool GEN, bool KO>
struct ColStager {
    using D = ColDims<P, TX, TY, TZ>;
    double pf[D::LZ];
    unsigned zo[D::LZ];                    // byte offset of plane q (uniform)
    const double *own;                     // field 0 of the block (uniform)
    long long fs;
    unsigned xy;                           // !GEN: byte offset of the column within a plane
    const double *below, *in, *above;      // GEN
    int qa;                                // GEN: first plane above the block (uniform)
    // interior column; column of the x or y stencils; column whose z sums the
    // mixed derivatives read (no corners: they are x or y stencils of them);
    // column that the x and y sums of a mixed field read besides
    bool ca, cf, cz, cm;

    __device__ __forceinline__ void setup(const StageArgs &a, const Tile &T, const z4c_block &B,
                                          unsigned t)
    {
        const int cx = t % D::LX, cy = t / D::LX, ng = B.ng;
        const int sy = B.nx + 2 * ng, sz = sy * (B.ny + 2 * ng);
        const bool inx = cx >= D::RAD && cx < D::RAD + TX, iny = cy >= D::RAD && cy < D::RAD + TY;
        ca = inx && iny;
        const bool cb = cx >= 1 && cx < D::LX - 1 && cy >= 1 && cy < D::LY - 1;
        cz = cb && (inx || iny);
        cf = KO ? (inx || iny) && cy < D::LY : cz;
        cm = cb || cf;
        own = a.u + B.offset;
        fs = B.field_stride;
        // ragged tiles: points beyond the stored region are clamped into it
        // (no active point's stencil reaches them)
        int gi = T.i0 - D::RAD + cx, gj = T.j0 - D::RAD + cy;
        gi = gi < B.nx + ng ? gi : B.nx + ng - 1;
        gj = gj < B.ny + ng ? gj : B.ny + ng - 1;
        const int ox = gi < 0 ? -1 : (gi >= B.nx ? 1 : 0);
        const int oy = gj < 0 ? -1 : (gj >= B.ny ? 1 : 0);
        const int wi = gi - ox * B.nx, wj = gj - oy * B.ny;   // wrapped
        const bool wrap = GEN || a.halo == Z4C_GHOST_PERIODIC;
#pragma unroll
        for (int q = 0; q < D::LZ; ++q) {
            int gk = T.k0 - D::RAD + q;
            gk = gk < B.nz + ng ? gk : B.nz + ng - 1;
            if (wrap)
                gk = gk < 0 ? gk + B.nz : (gk >= B.nz ? gk - B.nz : gk);
            zo[q] = 8u * (unsigned)((gk + ng) * sz);
        }
        const int stored = (gj + ng) * sy + gi + ng, wrapped = (wj + ng) * sy + wi + ng;
        if constexpr (!GEN) {
            xy = 8u * (unsigned)(wrap ? wrapped : stored);
        } else {
            auto source = [&](int oz) __attribute__((always_inline)) {
                if ((ox | oy | oz) == 0)
                    return own + stored;
                const int sb = a.halo == Z4C_GHOST_NEIGHBOUR
                    ? a.nbr[T.block * 27 + (oz + 1) * 9 + (oy + 1) * 3 + (ox + 1)] : -1;
                if (sb >= 0)   // same nx, ny, nz, ng and field stride as this block
                    return a.u + a.blocks[sb].offset + wrapped;
                // frozen, or the stored ghost that a refresh leaves as it is;
                // the plane offsets are wrapped ones
                return (a.frozen ? a.frozen + B.offset : own) + stored + (long long)(oz * B.nz) * sz;
            };
            in = source(0);
            below = T.k0 == 0 ? source(-1) : in;
            above = source(1);
            qa = B.nz - T.k0 + D::RAD;
        }
    }
    // Requests the points of field f that its stencils read.
    template <bool MIX>
    __device__ __forceinline__ void prefetch(int f)
    {
        auto load = [&](auto ld) __attribute__((always_inline)) {
            if (MIX ? cm : cf) {
#pragma unroll
                for (int q = D::RAD; q < D::RAD + TZ; ++q)
                    ld(q);
            }
            if (MIX ? cz : ca) {
#pragma unroll
                for (int q = 1; q < D::RAD; ++q) {
                    ld(q);
                    ld(D::LZ - 1 - q);
                }
            }
            if (KO && ca) {
                ld(0);
                ld(D::LZ - 1);
            }
        };
        if constexpr (GEN) {
            long long fo = f * fs * 8;
            // not formed for all fields at the start: the compiler kept 22 x 12
            // scalar sums in VGPR lanes (260 spilled, now 58); right-hand side of
            // one 64^3 block 79.8 -> 78.5 us, 8 x 40^3 radiative step 1.314 -> 1.302 ms
            asm volatile("" : "+s"(fo));
            typedef const __attribute__((address_space(1))) char gchar;
            gchar *const pb = (gchar *)below + fo, *const pi = (gchar *)in + fo,
                  *const pa = (gchar *)above + fo;
            load([&](int q) __attribute__((always_inline)) {
                gchar *p = q < D::RAD ? pb : (q < qa ? pi : pa);
                pf[q] = *(const gdouble *)(p + zo[q]);
            });
        } else {
            typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
            const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(own + (long long)f * fs), 0, -1, 0x00027000);
            load([&](int q) __attribute__((always_inline)) {
                const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rsrc, xy, zo[q], 0);
                pf[q] = __builtin_bit_cast(double, v);
            });
        }
    }
};

// First and second derivative and dissipation along one axis: the centre
// value and the taps c[0], c[ST], .. c[2 RAD ST] (centre at RAD ST).
template <int P, typename R, int ST>
__device__ __forceinline__ void axis(const double *c, double c0, R f1, R f2, R fk, R &d1, R &d2,
                                     R &ko)
{
    constexpr int RAD = P / 2 + 1;
    double p[5], m[5];
#pragma unroll
    for (int q = 1; q <= RAD; ++q) {
        p[q] = c[(RAD + q) * ST];
        m[q] = c[(RAD - q) * ST];
    }
    const double s1 = (p[1] - c0) + (m[1] - c0), s2 = (p[2] - c0) + (m[2] - c0),
                 s3 = (p[3] - c0) + (m[3] - c0);
    if constexpr (P == 4) {
        d1 = (R(8) * R(p[1] - m[1]) - R(p[2] - m[2])) * f1;
        d2 = (R(16) * R(s1) - R(s2)) * f2;
        ko = (R(15) * R(s1) - R(6) * R(s2) + R(s3)) * fk;
    } else {
        const double s4 = (p[4] - c0) + (m[4] - c0);
        d1 = (R(45) * R(p[1] - m[1]) - R(9) * R(p[2] - m[2]) + R(p[3] - m[3])) * f1;
        d2 = (R(270) * R(s1) - R(27) * R(s2) + R(2) * R(s3)) * f2;
        ko = (-R(56) * R(s1) + R(28) * R(s2) - R(8) * R(s3) + R(s4)) * fk;
    }
}

// Lopsided first derivative along one axis, unscaled (same 1/(c1 h) factor
// as the centred one): the order-P stencil on the points shifted by one
// towards the side `pos` (offsets -P/2+1 .. P/2+1 when pos, mirrored
// otherwise), in differences from the centre.  Weights, exact on
// polynomials of degree <= P: order 6 (2, -24, -35, 80, -30, 8, -1) / 60 at
// offsets -2 .. 4; order 4 (-3, -10, 18, -6, 1) / 12 at offsets -1 .. 3.
template <int P, typename R, int ST>
__device__ __forceinline__ R lopc(const double *c, double c0, bool pos)
{
    constexpr int RAD = P / 2 + 1;
    double a[P / 2 + 2], b[P / 2 + 2];   // a: the shifted side, b: the other
#pragma unroll
    for (int q = 1; q <= RAD; ++q) {
        const double pq = c[(RAD + q) * ST], mq = c[(RAD - q) * ST];
        a[q] = pos ? pq : mq;
        b[q] = pos ? mq : pq;
    }
    R v;
    if constexpr (P == 4)
        v = -R(3) * R(b[1] - c0) + R(18) * R(a[1] - c0) - R(6) * R(a[2] - c0) + R(a[3] - c0);
    else
        v = R(2) * R(b[2] - c0) - R(24) * R(b[1] - c0) + R(80) * R(a[1] - c0)
            - R(30) * R(a[2] - c0) + R(8) * R(a[3] - c0) - R(a[4] - c0);
    return pos ? v : -v;
}

// The staged field of a tile in LDS and this thread's view of it.
template <int P, int TX, int TY, int TZ, bool GEN, bool KO = true>
struct FieldTile {
    using D = ColDims<P, TX, TY, TZ>;
    using MZ = MixDimsZ<P, TX, TY, TZ>;
    ColStager<P, TX, TY, TZ, GEN, KO> st;
    double *pl, *zc, *zs, *ys;      // plane part, interior columns, z and y sums
    // LDS offsets of this thread (opaque to the compiler, so that they are
    // kept and not formed again for each field): its column in pl, zc and zs;
    // the lower corner of its x / y taps in pl and its row of y taps there (y
    // sums); where its y sum goes; its z and y sums
    unsigned t, pcol, zcol, zrow, po0, ysrc, ydst, pz, pz1, py;
    unsigned po, zo;                // taps in pl and zc, anew for each field
    bool ysum;

    __device__ __forceinline__ void setup(const StageArgs &a, const Tile &T, const z4c_block &B,
                                          unsigned thread, double *pl_, double *zc_, double *zs_,
                                          double *ys_)
    {
        t = thread;
        pl = pl_;
        zc = zc_;
        zs = zs_;
        ys = ys_;
        st.setup(a, T, B, t);
        const unsigned tx = t % TX, ty = (t / TX) % TY, tz = t / (TX * TY);
        const unsigned cx = t % D::LX, cy = t / D::LX;
        const unsigned sx = t % 16, sr = t / 16, ry = sr % TY, rz = sr / TY;
        pcol = cy * D::PX + cx;
        zcol = (cy - D::RAD) * TX + (cx - D::RAD);
        zrow = ((cy - 1) & 1) * MZ::ZR::OFF + ((cy - 1) >> 1) * 16 + cx - 1;
        po0 = tz * D::PLN + ty * D::PX + tx;
        ysum = sx < MZ::EX;
        ysrc = rz * D::PLN + (ry + D::RAD) * D::PX + sx + (D::RAD - MZ::Q);
        ydst = rz * MZ::YR::PLANE + (ry & 1) * MZ::YR::OFF + (ry >> 1) * 16 + sx;
        const unsigned r0 = ty + MZ::Q, r1 = r0 + 1;
        pz = tz * MZ::ZR::PLANE + (r0 & 1) * MZ::ZR::OFF + (r0 >> 1) * 16 + tx + MZ::Q;
        pz1 = tz * MZ::ZR::PLANE + (r1 & 1) * MZ::ZR::OFF + (r1 >> 1) * 16 + tx + MZ::Q;
        py = tz * MZ::YR::PLANE + (ty & 1) * MZ::YR::OFF + (ty >> 1) * 16 + tx + MZ::Q;
        asm volatile("" : "+v"(pcol), "+v"(zcol), "+v"(zrow), "+v"(po0), "+v"(ysrc), "+v"(ydst));
        asm volatile("" : "+v"(pz), "+v"(pz1), "+v"(py));
        po = po0;
        zo = t;
    }
    // Puts the requested field FF into LDS and requests field NX (-1: none).
    template <int FF, int NX, bool NAIVE = false>
    __device__ __forceinline__ void stage()
    {
        constexpr bool MIX = mixed_field(FF);
        __syncthreads();
        if constexpr (NAIVE) {
#pragma unroll
            for (int q = 0; q < D::LZ; ++q)
                st.pf[q] = double(float(st.pf[q]));
        }
        if (MIX ? st.cm : st.cf) {
#pragma unroll
            for (int z = 0; z < TZ; ++z)
                pl[z * D::PLN + pcol] = st.pf[D::RAD + z];
        }
        if (st.ca) {
#pragma unroll
            for (int q = KO ? 0 : 1; q < D::LZ - (KO ? 0 : 1); ++q)
                zc[q * TX * TY + zcol] = st.pf[q];
        }
        if constexpr (MIX) {
            if (st.cz) {
#pragma unroll
                for (int z = 0; z < TZ; ++z)
                    zs[z * MZ::ZR::PLANE + zrow] = d1raw<P, double, 1>(st.pf + z + D::RAD);
            }
        }
        if constexpr (NX >= 0)
            st.template prefetch<mixed_field(NX)>(NX);
        __syncthreads();
        if constexpr (MIX) {
            // y sums: 16 threads per row (those past EX idle)
            constexpr int NE = 16 * TY * TZ, DZ = D::NT / (16 * TY);
            static_assert(NE % D::NT == 0 && D::NT % (16 * TY) == 0, "whole planes per pass");
            if (ysum) {
#pragma unroll
                for (int q = 0; q < NE / D::NT; ++q)
                    ys[ydst + q * DZ * MZ::YR::PLANE] =
                        d1raw<P, double, D::PX>(pl + ysrc + q * DZ * D::PLN);
            }
            __syncthreads();
        }
        po = po0;
        zo = t;
        asm volatile("" : "+v"(po), "+v"(zo));
    }
    // Waits for the requested field's points.  Called by every lane before the
    // results of the staged field are stored: loads and stores are counted
    // together, so the wait at the next staging would be for those stores too.
    __device__ __forceinline__ void arrive()
    {
#pragma unroll
        for (int q = 0; q < D::LZ; ++q)
            asm volatile("" ::"v"(st.pf[q]));
    }
    // lowest taps of this thread's stencils, centre at RAD strides
    __device__ __forceinline__ const double *xtaps() const { return pl + po + D::RAD * D::PX; }
    __device__ __forceinline__ const double *ytaps() const { return pl + po + D::RAD; }
    __device__ __forceinline__ const double *ztaps() const { return zc + zo; }
    // value of the staged field at this thread's point
    __device__ __forceinline__ double centre() const { return pl[po + D::RAD * D::PX + D::RAD]; }
    // First and pure second derivatives and dissipation of the staged field.
    template <typename R>
    __device__ __forceinline__ void pure(const Fac<R> &F, R d[3], R &xx, R &yy, R &zz, R &ko) const
    {
        const double c0 = centre();
        R kx, ky, kz;
        axis<P, R, 1>(xtaps(), c0, F.d1[0], F.d2[0], F.ko[0], d[0], xx, kx);
        axis<P, R, D::PX>(ytaps(), c0, F.d1[1], F.d2[1], F.ko[1], d[1], yy, ky);
        axis<P, R, TX * TY>(ztaps(), c0, F.d1[2], F.d2[2], F.ko[2], d[2], zz, kz);
        ko = kx + ky + kz;
    }
    // The same with the lopsided first derivatives l for a shift `beta`, an axis
    // finished before the taps of the next are read: with those of all three axes
    // in flight the compiler spilled values that live through the whole kernel,
    // and each reload waited behind the next field's points (ragged blocks of
    // 20/13/33 x 19 points 494 us, so 424).
    template <typename R>
    __device__ __forceinline__ void pure_lopsided(const Fac<R> &F, const R beta[3], R d[3], R &xx,
                                                  R &yy, R &zz, R &ko, R l[3]) const
    {
        const double c0 = centre();
        R kx, ky, kz;
        axis<P, R, 1>(xtaps(), c0, F.d1[0], F.d2[0], F.ko[0], d[0], xx, kx);
        l[0] = lopc<P, R, 1>(xtaps(), c0, beta[0] > R(0)) * F.d1[0];
        __builtin_amdgcn_sched_barrier(0);
        axis<P, R, D::PX>(ytaps(), c0, F.d1[1], F.d2[1], F.ko[1], d[1], yy, ky);
        l[1] = lopc<P, R, D::PX>(ytaps(), c0, beta[1] > R(0)) * F.d1[1];
        __builtin_amdgcn_sched_barrier(0);
        axis<P, R, TX * TY>(ztaps(), c0, F.d1[2], F.d2[2], F.ko[2], d[2], zz, kz);
        l[2] = lopc<P, R, TX * TY>(ztaps(), c0, beta[2] > R(0)) * F.d1[2];
        __builtin_amdgcn_sched_barrier(0);
        ko = kx + ky + kz;
    }
    // Mixed second derivatives, from the sums (formed in double also for
    // float arithmetic: a difference of rounded sums would lose digits).
    template <typename R>
    __device__ __forceinline__ void mixed(const Fac<R> &F, R dd[6]) const
    {
        dd[1] = R(d1sum<P, double, 1>(ys + py)) * F.mix[0];
        dd[2] = R(d1sum<P, double, 1>(zs + pz)) * F.mix[1];
        dd[4] = R(d1sum_rows<P, double>(zs + pz, zs + pz1)) * F.mix[2];
    }
};

}  // namespace tile

// Launches: halo sources beyond the block itself only under the frozen and
// neighbour rules.
inline bool general_halo(const StageArgs &a)
{
    return a.halo == Z4C_GHOST_FROZEN || a.halo == Z4C_GHOST_NEIGHBOUR;
}

}  // namespace z4c
