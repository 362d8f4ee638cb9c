// z4c_matter.hip -- matter coupling of the Z4c right-hand side: Lagrange
// interpolation between the vertex-centred Z4c grid and the cell-centred
// fluid grid (Sec. 3.2, intergrid communication) and the ADM projections of
// the perfect-fluid / ideal-GRMHD stress-energy tensor (Sec. 2.1, 2.2).
//
// Interpolation is separable and marches along z: a workgroup of 256
// threads owns a column of w x h outputs and d output planes of one field (even
// shares of a block, chosen when the plan is made); for each input plane it stages
// the (w + order - 1)(h + order - 1) inputs in LDS (the next planes already in
// flight in registers), reduces them along x and then y, and each thread keeps
// the y-reduced values of the last `order` planes in registers for the z
// reduction, so every input plane is read once per column and the z halo costs
// order - 1 planes in d.  The ADM projections are
// pointwise, one cell per thread over contiguous chunks of stored cells.
// Both kernels are HBM-bound.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "z4c_internal.h"
#include "z4c_matter.h"

struct z4c_mplan {
    std::vector<z4c_mblock> blocks;
    bool device = false;
    z4c_mblock *blocks_d = nullptr;
    void *cc_tiles_d = nullptr;   // ITile[n_cc]: interpolation columns over every stored cell
    void *vc_tiles_d = nullptr;   // ITile[n_vc]: interpolation columns over vertices [0, nc]
    void *pt_tiles_d = nullptr;   // MTile[n_pt]: point tiles over every stored cell
    int n_cc = 0, n_vc = 0, n_pt = 0;
};

namespace z4c {
namespace {

constexpr int INT_ = 256;   // threads of an interpolation workgroup
// ADM projections: chunks of PNT consecutive stored cells, one per thread
constexpr int PNT = 512;

struct MTile {
    int block, i0;   // chunk of stored cells from linear index i0
};

// Column of an interpolation: outputs [i0, i0 + w) x [j0, j0 + h) x
// [k0, k0 + d) of the call's range, one thread per (x, y).
struct ITile {
    int block, i0, j0, k0, w, h, d;
};

// Buffer size and the byte offset of outputs that are not stored; a column's
// rows span less.
constexpr unsigned OUTSIDE = 0xfffffff0u;

// Weight k of the Lagrange polynomial through O equally spaced nodes,
// evaluated midway between the two central nodes.
template <int O>
__device__ __forceinline__ constexpr double midw(int k)
{
    if constexpr (O == 2)
        return 0.5;
    else if constexpr (O == 4)
        return (k == 0 || k == 3) ? -1.0 / 16.0 : 9.0 / 16.0;
    else
        return (k == 0 || k == 5) ? 3.0 / 256.0 : ((k == 1 || k == 4) ? -25.0 / 256.0 : 150.0 / 256.0);
}

template <int O>
__device__ __forceinline__ double midsum(const double *c, int st)
{
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < O; ++k)
        s += midw<O>(k) * c[k * st];
    return s;
}

// Interpolates fields [f0, f0 + nf) of one column, f0 = (logical workgroup / n)
// nf: TO_CC the 7 conformal-geometry fields of the VC state to cells (stored CC
// index in [ngc - ext, ngc + nc + ext)); otherwise the 10 ADM fields from the
// CC sources to vertices [0, nc].
// Each input plane goes through LDS and its x sums through LDS again; the last
// O y sums of a column stay in registers.  Both LDS arrays are double-buffered,
// so that the x sums of a plane and the y and z sums of the one before it share
// one barrier interval.  Loads and stores take no branch (positions outside are
// clamped into the stored array and feed no output of the range; stores outside
// it fall to the buffer's bounds check): the wait for a plane then counts what
// was issued after it and leaves the younger planes in flight.
// What bounds it: HBM, at 3.7 to 4.3 TB/s of reads and writes, every point once
// (1.51 + 1.40 GB for the 10 fields of 8 x 128^3 cells at order 6).  Against
// 32 x 8 x 16 columns with two barriers per plane and the fields in a loop:
// 1090 -> 783 us, the 7 metric fields at order 4 674 -> 557 us, and 8 x 20^3
// cells 81 -> 10 and 47 -> 9 us.  Four waves per SIMD (all that fit: 902 and 674
// us where four took 856 and 660).  The fields of a column one after the other
// in one workgroup 1016 us, side by side on one XCD 1047 us.
template <int O, bool TO_CC>
__global__ void __launch_bounds__(INT_)
    __attribute__((amdgpu_waves_per_eu(4, 4)))
interp_kernel(const z4c_mblock *blocks, const ITile *tiles, int n, int nf, int ext,
              const double *in, double *out)
{
    constexpr int PD = O == 6 ? 6 : 4;   // planes in flight; a multiple of O and of 2
    constexpr int NLD = 2;               // values of an input plane per thread
    __shared__ __attribute__((aligned(16))) double s_pl[2][NLD * INT_ + 4];
    __shared__ __attribute__((aligned(16))) double s_x[2][2 * INT_];
    const int wg = xcd_logical(blockIdx.x, gridDim.x);
    const ITile T = tiles[wg % n];
    const z4c_mblock B = blocks[T.block];
    const int nc[3] = {B.ncx, B.ncy, B.ncz}, o[3] = {T.i0, T.j0, T.k0};
    // per direction: outputs left in the range, stored index of output 0 and
    // of its first input, stored extents
    int left[3], out0[3], in0[3], is[3], os[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int vc = nc[d] + 1 + 2 * B.ngv, cc = nc[d] + 2 * B.ngc;
        left[d] = (TO_CC ? nc[d] + 2 * ext : nc[d] + 1) - o[d];
        out0[d] = o[d] + (TO_CC ? B.ngc - ext : B.ngv);
        in0[d] = o[d] - O / 2 + (TO_CC ? B.ngv + 1 - ext : B.ngc);
        is[d] = TO_CC ? vc : cc;
        os[d] = TO_CC ? cc : vc;
    }
    if (left[0] <= 0 || left[1] <= 0 || left[2] <= 0)
        return;   // outside this call's range (uniform)
    const int nz = T.d < left[2] ? T.d : left[2];
    const unsigned t = threadIdx.x;
    // input plane: this thread's values, their offsets and LDS places (rows
    // padded to an even length)
    const unsigned lx = T.w + O - 1, ly = T.h + O - 1, lxp = (lx + 1) & ~1u;
    long long ioff[NLD];
    unsigned place[NLD];
#pragma unroll
    for (int q = 0; q < NLD; ++q) {
        const unsigned e = t + q * INT_, y = e / lx, x = e - y * lx;
        const int gx = min(max(in0[0] + (int)x, 0), is[0] - 1);
        const int gy = min(max(in0[1] + (int)y, 0), is[1] - 1);
        ioff[q] = gx + (long long)is[0] * gy;
        place[q] = y < ly ? y * lxp + x : NLD * INT_ + 2;
    }
    // x sums of two neighbouring outputs of row xr
    const unsigned pw = (T.w + 1) / 2, xr = t / pw, xp = t - xr * pw;
    const bool xsum = xr < ly;
    const unsigned xsrc = xr * lxp + 2 * xp, xdst = 2 * t;
    // this thread's column; past the buffer's end where it has no output
    const unsigned ty = t / T.w, tx = t - ty * T.w;
    const unsigned ysrc = (ty < (unsigned)T.h ? ty : T.h - 1) * 2 * pw + tx;
    const bool ok = ty < (unsigned)T.h && (int)tx < left[0] && (int)ty < left[1];
    const unsigned ooff = ok ? 8u * (tx + (unsigned)os[0] * ty) : OUTSIDE;
    const long long ips = (long long)is[0] * is[1], ops = (long long)os[0] * os[1];
    const int np = nz + O - 1;   // input planes of the column

    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const int fe = TO_CC ? 7 : 10, f0 = wg / n * nf, f1 = f0 + nf < fe ? f0 + nf : fe;
    for (int f = f0; f < f1; ++f) {
        const double *src = in + (TO_CC ? B.vs_offset + f * B.vc_stride
                                        : B.ca_offset + f * B.cc_stride);
        double *dst = out + (TO_CC ? B.cg_offset + f * B.cc_stride : B.vm_offset + f * B.vc_stride)
                    + out0[0] + (long long)os[0] * out0[1] + out0[2] * ops;
        double r[PD][NLD];   // planes p .. p + PD - 1
        auto load = [&](int j, int p) __attribute__((always_inline)) {
            const int z = min(max(in0[2] + min(p, np - 1), 0), is[2] - 1);
            const double *c = src + z * ips;
#pragma unroll
            for (int q = 0; q < NLD; ++q)
                r[j][q] = c[ioff[q]];
        };
#pragma unroll
        for (int p = 0; p < PD; ++p)
            load(p, p);
        double col[O];   // y sums of the last O planes, plane p in col[p % O]
#pragma unroll
        for (int k = 0; k < O; ++k)
            col[k] = 0.0;
        for (int p0 = 0;; p0 += PD) {
#pragma unroll
            for (int j = 0; j < PD; ++j) {
                const int p = p0 + j;
                if (p > np)
                    goto done;
#pragma unroll
                for (int q = 0; q < NLD; ++q)
                    s_pl[j & 1][place[q]] = r[j][q];
                load(j, p + PD);
                __syncthreads();
                if (xsum) {
                    const double2 *c = (const double2 *)(s_pl[j & 1] + xsrc);
                    double v[O + 2];
#pragma unroll
                    for (int k = 0; k < O + 2; k += 2) {
                        const double2 w = c[k / 2];
                        v[k] = w.x;
                        v[k + 1] = w.y;
                    }
                    *(double2 *)(s_x[j & 1] + xdst) =
                        make_double2(midsum<O>(v, 1), midsum<O>(v + 1, 1));
                }
                // plane p - 1; output plane p - O, below the range at first
                constexpr int M = PD - 1;
                col[(j + M) % O] = midsum<O>(s_x[(j + 1) & 1] + ysrc, 2 * pw);
                double v = 0.0;
#pragma unroll
                for (int k = 0; k < O; ++k)
                    v += midw<O>(k) * col[(j + M + 1 + k) % O];
                const auto plane = __builtin_amdgcn_make_buffer_rsrc(
                    (void *)(dst + (p - O) * ops), 0, p >= O ? (int)OUTSIDE : 0, 0x00027000);
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), plane, ooff, 0,
                                                      0);
            }
        }
    done:
        __syncthreads();   // the LDS arrays are written again by the next field
    }
}

// ADM projections at the cells of one tile (stored CC index in
// [ngc - ext, ngc + nc + ext)).
template <bool MHD>
__global__ void __launch_bounds__(PNT)
adm_kernel(const z4c_mblock *blocks, const MTile *tiles, int ext, double gfac, double chi_floor,
           const double *geom, const double *prim, double *adm)
{
    const MTile T = tiles[blockIdx.x];
    const z4c_mblock B = blocks[T.block];
    const int sx = B.ncx + 2 * B.ngc, sy = B.ncy + 2 * B.ngc;
    const long long fs = B.cc_stride;
    const int a0 = B.ngc - ext;
    const int ax = B.ngc + B.ncx + ext, ay = B.ngc + B.ncy + ext, az = B.ngc + B.ncz + ext;
    {
        // T.i0: first stored cell (linear index) of the chunk
        const long long lin = (long long)T.i0 + threadIdx.x;
        if (lin >= (long long)sx * sy * (B.ncz + 2 * B.ngc))
            return;
        const int x = (int)(lin % sx), r = (int)(lin / sx), y = r % sy, z = r / sy;
        if (x < a0 || y < a0 || z < a0 || x >= ax || y >= ay || z >= az)
            return;
        const long long p = lin;
        const double *g = geom + B.cg_offset + p;
        const double *w = prim + B.cp_offset + p;
        const double chi = g[0];
        const double ic = 1.0 / (chi > chi_floor ? chi : chi_floor);
        double gam[6];
#pragma unroll
        for (int q = 0; q < 6; ++q)
            gam[q] = g[(1 + q) * fs] * ic;
        const double rho = w[0], ux = w[fs], uy = w[2 * fs], uz = w[3 * fs], pr = w[4 * fs];
        // ut_i = gamma_ij ut^j
        const double lx = gam[0] * ux + gam[1] * uy + gam[2] * uz;
        const double ly = gam[1] * ux + gam[3] * uy + gam[4] * uz;
        const double lz = gam[2] * ux + gam[4] * uy + gam[5] * uz;
        const double W = sqrt(1.0 + lx * ux + ly * uy + lz * uz);
        const double iW = 1.0 / W;
        const double v[3] = {lx * iW, ly * iW, lz * iW};   // v_i
        const double rhoh = rho + gfac * pr;
        double E, P, ab0 = 0.0, b[3] = {0.0, 0.0, 0.0};
        if constexpr (MHD) {
            const double Bx = w[5 * fs], By = w[6 * fs], Bz = w[7 * fs];
            const double Blx = gam[0] * Bx + gam[1] * By + gam[2] * Bz;
            const double Bly = gam[1] * Bx + gam[3] * By + gam[4] * Bz;
            const double Blz = gam[2] * Bx + gam[4] * By + gam[5] * Bz;
            ab0 = W * (Bx * v[0] + By * v[1] + Bz * v[2]);           // alpha b^0
            const double B2 = Blx * Bx + Bly * By + Blz * Bz;
            const double b2 = (ab0 * ab0 + B2) * iW * iW;
            b[0] = Blx * iW + ab0 * v[0];                             // b_i
            b[1] = Bly * iW + ab0 * v[1];
            b[2] = Blz * iW + ab0 * v[2];
            E = (rhoh + b2) * W * W;
            P = pr + 0.5 * b2;
        } else {
            E = rhoh * W * W;
            P = pr;
        }
        double *o = adm + B.ca_offset + p;
        o[0] = E - P - ab0 * ab0;
#pragma unroll
        for (int i = 0; i < 3; ++i)
            o[(1 + i) * fs] = E * v[i] - ab0 * b[i];
        constexpr int QI[6] = {0, 0, 0, 1, 1, 2}, QJ[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
        for (int q = 0; q < 6; ++q)
            o[(4 + q) * fs] = E * v[QI[q]] * v[QJ[q]] + P * gam[q] - b[QI[q]] * b[QJ[q]];
    }
}

// ---- primitive <-> conservative maps (ideal gas, Sec. 2.2; Appendix A) ----

struct C2PArgs {
    const z4c_mblock *blocks;
    const MTile *tiles;
    int ext, mhd, max_iter;
    double gm1, chi_floor, rho_atm, p_atm, eps_atm, rho_thr, vmax2, ut_max2, tol, newton_tol, g_tol;
    const double *geom;
    const double *prim_in;    // p2c
    double *cons;
    double *prim;             // c2p
    int *status;
};

// Cell of one thread (chunk of consecutive stored cells) or -1 when it lies
// outside [ngc - ext, ngc + nc + ext) per direction.
__device__ __forceinline__ long long chunk_cell(const z4c_mblock &B, const MTile &T, int ext)
{
    // a block has at most 2^31 - 1 stored cells
    const unsigned sx = B.ncx + 2 * B.ngc, sy = B.ncy + 2 * B.ngc;
    const unsigned lin = (unsigned)T.i0 + threadIdx.x;
    if (lin >= sx * sy * (unsigned)(B.ncz + 2 * B.ngc))
        return -1;
    const unsigned r = lin / sx, zz = r / sy;
    const int x = (int)(lin - r * sx), y = (int)(r - zz * sy), z = (int)zz;
    const int a0 = B.ngc - ext;
    if (x < a0 || y < a0 || z < a0 || x >= B.ngc + B.ncx + ext || y >= B.ngc + B.ncy + ext
        || z >= B.ngc + B.ncz + ext)
        return -1;
    return lin;
}

// gamma_ij (6, symmetric storage) from the CC geometry, its determinant.
__device__ __forceinline__ double cell_metric(const double *g, long long fs, double chi_floor,
                                              double gam[6])
{
    const double chi = g[0];
    const double ic = 1.0 / (chi > chi_floor ? chi : chi_floor);
#pragma unroll
    for (int q = 0; q < 6; ++q)
        gam[q] = g[(1 + q) * fs] * ic;
    return gam[0] * (gam[3] * gam[5] - gam[4] * gam[4]) - gam[1] * (gam[1] * gam[5] - gam[4] * gam[2])
         + gam[2] * (gam[1] * gam[4] - gam[3] * gam[2]);
}

__device__ __forceinline__ void lower(const double gam[6], const double u[3], double l[3])
{
    l[0] = gam[0] * u[0] + gam[1] * u[1] + gam[2] * u[2];
    l[1] = gam[1] * u[0] + gam[3] * u[1] + gam[4] * u[2];
    l[2] = gam[2] * u[0] + gam[4] * u[1] + gam[5] * u[2];
}

// Conservatives (densitised) of rho, ut^i, p, B^i.  With W^2 = 1 + ut.ut,
// v_i = ut_i / W, alpha b^0 = W B.v, b_i = B_i / W + alpha b^0 v_i,
// b^2 = ((alpha b^0)^2 + B^2) / W^2 (the lapse cancels):
//   D = sg rho W,  S_j = sg ((rho h + b^2) W ut_j - alpha b^0 b_j),
//   tau = sg ((rho h + b^2) W^2 - rho W - (p + b^2/2) - (alpha b^0)^2).
template <bool MHD>
__device__ __forceinline__ void p2c_point(const double gam[6], double sg, double gm1, double rho,
                                          const double ut[3], double p, const double Bu[3],
                                          double q[8])
{
    double ul[3];
    lower(gam, ut, ul);
    const double W2 = 1.0 + ul[0] * ut[0] + ul[1] * ut[1] + ul[2] * ut[2];
    const double W = sqrt(W2);
    const double rhoh = rho + (1.0 + 1.0 / gm1) * p;   // rho (1 + eps) + p
    double ab0 = 0.0, b2 = 0.0, bl[3] = {0.0, 0.0, 0.0};
    if constexpr (MHD) {
        double Bl[3];
        lower(gam, Bu, Bl);
        const double iW = 1.0 / W;
        ab0 = (Bu[0] * ul[0] + Bu[1] * ul[1] + Bu[2] * ul[2]);         // W B.v = B.ut
        b2 = (ab0 * ab0 + Bl[0] * Bu[0] + Bl[1] * Bu[1] + Bl[2] * Bu[2]) * iW * iW;
#pragma unroll
        for (int i = 0; i < 3; ++i)
            bl[i] = Bl[i] * iW + ab0 * ul[i] * iW;                        // v_i = ut_i / W
    }
    const double e = rhoh + b2;
    q[0] = sg * rho * W;
#pragma unroll
    for (int i = 0; i < 3; ++i)
        q[1 + i] = sg * (e * W * ul[i] - ab0 * bl[i]);
    q[4] = sg * (e * W2 - rho * W - (p + 0.5 * b2) - ab0 * ab0);
    if constexpr (MHD) {
#pragma unroll
        for (int i = 0; i < 3; ++i)
            q[5 + i] = sg * Bu[i];
    }
}

template <bool MHD>
__global__ void __launch_bounds__(PNT) p2c_kernel(const C2PArgs a)
{
    const MTile T = a.tiles[blockIdx.x];
    const z4c_mblock B = a.blocks[T.block];
    const long long p = chunk_cell(B, T, a.ext);
    if (p < 0)
        return;
    const long long fs = B.cc_stride;
    double gam[6];
    const double sg = sqrt(cell_metric(a.geom + B.cg_offset + p, fs, a.chi_floor, gam));
    const double *w = a.prim_in + B.cp_offset + p;
    const double ut[3] = {w[fs], w[2 * fs], w[3 * fs]};
    double Bu[3] = {0.0, 0.0, 0.0};
    if constexpr (MHD) {
        Bu[0] = w[5 * fs];
        Bu[1] = w[6 * fs];
        Bu[2] = w[7 * fs];
    }
    double q[8];
    p2c_point<MHD>(gam, sg, a.gm1, w[0], ut, w[4 * fs], Bu, q);
    double *o = a.cons + B.cq_offset + p;
    constexpr int NQ = MHD ? 8 : 5;
#pragma unroll
    for (int i = 0; i < NQ; ++i)
        o[i * fs] = q[i];
}

// Primitive recovery of one cell: the master function of Kastaun, Kalinani &
// Ciolfi in mu = 1 / (h W), with the normalised conservatives q = tau / D,
// r_i = S_i / D, b^i = B^i / sqrt(D) (all undensitised):
//   x = 1 / (1 + mu b^2),  rbar^2 = x^2 r^2 + mu x (1 + x) (r.b)^2,
//   qbar = q - b^2/2 - mu^2 x^2 (b^2 r^2 - (r.b)^2) / 2,
//   v^2 = min(mu^2 rbar^2, vmax^2),  W = 1 / sqrt(1 - v^2),  rho = D / W,
//   eps = max(W (qbar - mu rbar^2) + v^2 W^2 / (1 + W), 0),
//   a = p / (rho (1 + eps)),  h = (1 + eps)(1 + a),
//   nu = max(h / W, (1 + a)(1 + qbar - mu rbar^2)),  mu_hat = 1 / (nu + mu rbar^2),
//   f(mu) = mu - mu_hat(mu).
// For the ideal gas p = (Gamma - 1) rho eps this reduces exactly to
//   eps = max(W (qbar - mu rbar^2 + 1) - 1, 0)   (v^2 W^2 / (1 + W) = W - 1),
//   h = 1 + Gamma eps,  nu = h / W            (the two branches of the max
//   coincide unless eps is clamped, when h / W is the larger),
// and, nu + mu rbar^2 being positive, the root and the sign of f are those
// of g(mu) = mu (nu + mu rbar^2) - 1, which needs no division.
// The function's derivative is cheap beside it: with C = b^2 r^2 - (r.b)^2,
// d rbar^2 / d mu = -2 x^3 C, d qbar / d mu = -mu x^3 C, so that
// s = qbar - mu rbar^2 + 1 has s' = mu x^3 C - rbar^2 and
// nu' = s' (Gamma - (Gamma - 1) mu W) (mu W s' where eps is clamped).
// What a root is worth is set by the rounding of one evaluation near it: errors
// of mu^2 rbar^2 count W^2 times, those of qbar b^2 / D times (its terms cancel),
// and those of the unit parts of s, 1 / W, D and mu as much as the rest where the
// gas is slow and cold.  The products, mu x and b^2 r^2 - (r.b)^2 carry their
// rounding errors along and the units are kept apart, some dozen fused operations;
// one Newton result is then more exact than a bracket shrunk around a sign change
// of the plain expressions (rms error of mu against 113-bit roots: W < 2 without
// field 2.1e-16 -> 0.6e-16, W < 19 2.4e-16 -> 1.8e-16, b^2 / rho = 1 .. 10
// 4.9e-16 -> 2.2e-16, 10^4 1.1e-12 -> 3.1e-16), where the plain expressions' Newton
// result was less with a field (6.2e-16 and 1.7e-12).
template <bool MHD>
struct Master {
    double q, r2, b2, rb2, gam, vmax2;
    double C, Cl, a0, a0l;   // b^2 r^2 - (r.b)^2 and q - b^2/2, value and remainder

    __device__ __forceinline__ static double diff_error(double a, double b, double d)
    {
        const double bb = a - d;   // d = a - b rounded; the exact remainder
        return (a - (d + bb)) + (bb - b);
    }
    __device__ __forceinline__ void prepare()
    {
        if constexpr (MHD) {
            const double p = b2 * r2;
            C = p - rb2;
            Cl = diff_error(p, rb2, C) + fma(b2, r2, -p);
            a0 = q - 0.5 * b2;
            a0l = diff_error(q, 0.5 * b2, a0);
            if (!(C < INFINITY)) {   // b^2 r^2 beyond double: qbar is -infinity
                a0 = -C;
                C = Cl = a0l = 0.0;
            }
        }
    }
    __device__ __forceinline__ double x(double mu) const { return MHD ? 1.0 / (1.0 + mu * b2) : 1.0; }
    __device__ __forceinline__ double rbar2(double mu) const
    {
        if constexpr (!MHD)
            return r2;
        const double xx = x(mu);
        return r2 * xx * xx + mu * xx * (1.0 + xx) * rb2;
    }
    // 1 / v to a few parts in 10^15: for a factor whose error is carried along or
    // which scales a small correction
    __device__ __forceinline__ static double inverse(double v)
    {
        const double i = __builtin_amdgcn_rcp(v);
        return fma(fma(-v, i, 1.0), i, i);
    }
    // x, rbar^2, s = qbar - mu rbar^2 and t = 1 - mu^2 rbar^2 at mu
    struct At {
        double x, rb, s, t;
    };
    __device__ __forceinline__ At at(double mu) const
    {
        At e;
        double qb = q, ql = 0.0;
        if constexpr (MHD) {
            const double d = fma(mu, b2, 1.0), dl = fma(mu, b2, 1.0 - d);   // 1 - d is exact
            double x = inverse(d);
            x = fma(fma(-d, x, 1.0), x, x);
            e.x = x;
            const double y = mu * x;
            const double yl = fma(-y, dl, fma(-y, d, mu)) * x;   // mu / (1 + mu b^2) - y
            const double Cy = C * y, Cyl = fma(Cl, y, fma(C, y, -Cy));
            qb = fma(-0.5 * Cy, y, a0);
            ql = fma(-Cy, yl, fma(-0.5 * y, Cyl, a0l));
            e.rb = r2 * e.x * e.x + y * (1.0 + e.x) * rb2;
        } else {
            e.x = 1.0;
            e.rb = r2;
        }
        e.s = fma(-mu, e.rb, qb) + ql;
        const double p = mu * e.rb;
        e.t = fma(-p, mu, 1.0) - fma(mu, e.rb, -p) * mu;
        return e;
    }
    // D - 1, D = nu + mu rbar^2, from iw = 1 / W - 1: nu is 1 / W where eps is
    // clamped, else Gamma (1 + s) - (Gamma - 1) / W.
    __device__ __forceinline__ double d1(double mu, const At &p, double iw) const
    {
        return fma(mu, p.rb, p.s > iw ? fma(gam, p.s, -(gam - 1.0) * iw) : iw);
    }
    // Whether g(0) is -1 and not a NaN, as 0 D is from an infinite D (r^2, b^2 or
    // q beyond double): such a cell has no sign change.
    __device__ __forceinline__ bool starts() const
    {
        return r2 < INFINITY && b2 < INFINITY && rb2 < INFINITY
            && !(gam * (q - 0.5 * b2) >= INFINITY);
    }
    // g = mu D - 1; the unit parts of mu and D meet without a rounding
    __device__ __forceinline__ static double residual(double mu, double D1)
    {
        const double m = mu - 1.0;
        return fma(mu, D1, m) + (mu - (m + 1.0));
    }
    // g(mu); W and eps of the estimate
    __device__ __forceinline__ double f(double mu, double &W, double &eps) const
    {
        const At p = at(mu);
        const double t = fmax(p.t, 1.0 - vmax2), r = rsqrt(t), w = t * r;
        const double iW = fma(0.5 * r, fma(-w, w, t), w), iw = iW - 1.0;
        W = fma(r, fma(-iW, r, 1.0), r);
        eps = p.s > iw ? W * (p.s - iw) : 0.0;
        return residual(mu, d1(mu, p, iw));
    }
    // g(mu), the Newton step of f(mu) = mu - 1 / D, f / f' = D g / (D^2 + D'), and
    // the iterate it leads to, from f without cancellation where the step is long
    // (mu+ may be any factor above the root of a hot cell).
    __device__ __forceinline__ double newton(double mu, double &step, double &next) const
    {
        const At p = at(mu);
        const double mx3C = MHD ? mu * p.x * p.x * p.x * C : 0.0;
        const bool fast = !(p.t >= 1.0 - vmax2);
        const double t = fast ? 1.0 - vmax2 : p.t;
        const double W = rsqrt(t), w = t * W, iw = fma(0.5 * W, fma(-w, w, t), w) - 1.0;
        const double D1 = d1(mu, p, iw), D = 1.0 + D1, g = residual(mu, D1);
        const double sp = mx3C - p.rb, mW = fast ? 0.0 : mu * W;
        const double Dp = sp * (p.s > iw ? gam - (gam - 1.0) * mW : mW) + p.rb - 2.0 * mx3C;
        const double den = D * D + Dp;
        // the step needs few digits of its own: the iterate it leads to is
        // wrong by their error times the step
        step = D * g * inverse(den);
        next = mu - step;
        if (!(fabs(step) < 0.5 * mu)) {
            const double r = Dp / D;
            next = (1.0 + mu * r) / (D + r);
            step = mu - next;
        }
        return g;
    }
    // The root mu+ of mu sqrt(1 + rbar^2(mu)) - 1 (minimum enthalpy 1), by
    // Newton's method on S = mu^2 (1 + rbar^2) - 1; rbar^2 decreases with mu,
    // so the root lies between 1 / sqrt(1 + rbar^2) at mu = 0 and at mu = 1.
    // The lower end of the last bracket would cut the root off, its upper end
    // (returned when the iteration is not done after a few steps) does not.
    __device__ __forceinline__ double mu_plus() const
    {
        double hi = 1.0 / sqrt(1.0 + rbar2(1.0));
        if constexpr (!MHD) {   // the root itself: mu^2 (1 + r^2) = 1
            const double p = hi * r2;
            return fma(0.5 * hi, fma(-p, hi, 1.0) - fma(hi, hi, fma(hi, r2, -p) * hi), hi);
        }
        double lo = 1.0 / sqrt(1.0 + r2), mu = hi;
        for (int it = 0; it < 10 && hi - lo > 1e-15; ++it) {
            const double xx = x(mu);
            const double h = 1.0 + r2 * xx * xx + mu * xx * (1.0 + xx) * rb2;
            const double v = mu * mu * h - 1.0;
            const double d = v * inverse(2.0 * mu * (h - mu * xx * xx * xx * C));
            if (v > 0.0)
                hi = mu;
            else
                lo = mu;
            const double m = mu - d;
            const bool in = m > lo && m < hi;
            mu = in ? m : 0.5 * (lo + hi);
            if (in ? fabs(d) <= 1e-9 * mu : d == 0.0)
                return mu;
        }
        return hi;
    }
};

// Illinois iterations for a sign change of fn on [lo, hi] (fn(lo) < 0 <=
// fn(hi)), every eighth step a bisection (the bracket shrinks whatever fn
// does): what a cell whose Newton steps take too long falls back to.
// Converged when the bracket is narrower than tol * hi or one ulp; returns
// false after max_iter steps without convergence.  An end where fn is
// exactly zero is the root.
template <typename Fn>
__device__ __forceinline__ bool illinois(Fn fn, double lo, double hi, double flo, double fhi,
                                         double tol, int max_iter, double &root)
{
    if (fhi == 0.0 || flo == 0.0) {
        root = fhi == 0.0 ? hi : lo;
        return true;
    }
    int side = 0;
    for (int it = 0; it < max_iter; ++it) {
        double m = (lo * fhi - hi * flo) / (fhi - flo);
        if (!(m > lo && m < hi) || (it & 7) == 7)
            m = 0.5 * (lo + hi);
        if (!(m > lo && m < hi)) {
            root = m;
            return true;
        }
        const double fm = fn(m);
        if (fm == 0.0) {
            root = m;
            return true;
        }
        if (fm < 0.0) {
            lo = m;
            flo = fm;
            if (side == -1)
                fhi *= 0.5;
            side = -1;
        } else {
            hi = m;
            fhi = fm;
            if (side == 1)
                flo *= 0.5;
            side = 1;
        }
        if (hi - lo <= tol * hi) {
            root = 0.5 * (lo + hi);
            return true;
        }
    }
    return false;
}

// Primitive recovery, one cell per thread.  A wave runs its slowest lane's
// iterations: Illinois steps for mu+ and for the root took 24 evaluations per
// wave and bound the kernel by FP64 arithmetic (1.81 ms for 8.5 M cells of a
// magnetised star and its atmosphere); Newton steps take 2 + 3, and it is
// bound by HBM (0.383 ms, 4.1 of the 4.85 TB/s a large copy reaches).
template <bool MHD>
__global__ void __launch_bounds__(PNT) c2p_kernel(const C2PArgs a)
{
    const MTile T = a.tiles[blockIdx.x];
    const z4c_mblock B = a.blocks[T.block];
    const long long p = chunk_cell(B, T, a.ext);
    if (p < 0)
        return;
    const long long fs = B.cc_stride;
    double gam[6];
    const double det = cell_metric(a.geom + B.cg_offset + p, fs, a.chi_floor, gam);
    const double sg = sqrt(det), isg = 1.0 / sg;
    double *c = a.cons + B.cq_offset + p;
    const double D = c[0] * isg;
    const double Sl[3] = {c[fs] * isg, c[2 * fs] * isg, c[3 * fs] * isg};
    const double tau = c[4 * fs] * isg;
    double Bu[3] = {0.0, 0.0, 0.0};
    if constexpr (MHD) {
        Bu[0] = c[5 * fs] * isg;
        Bu[1] = c[6 * fs] * isg;
        Bu[2] = c[7 * fs] * isg;
    }
    int st = 0;
    double rho = 0.0, pr = 0.0, ut[3] = {0.0, 0.0, 0.0};
    if (!(D >= a.rho_thr)) {
        st = 1;
    } else {
        // inverse metric
        const double id = 1.0 / det;
        const double gi[6] = {(gam[3] * gam[5] - gam[4] * gam[4]) * id,
                              (gam[2] * gam[4] - gam[1] * gam[5]) * id,
                              (gam[1] * gam[4] - gam[2] * gam[3]) * id,
                              (gam[0] * gam[5] - gam[2] * gam[2]) * id,
                              (gam[2] * gam[1] - gam[0] * gam[4]) * id,
                              (gam[0] * gam[3] - gam[1] * gam[1]) * id};
        const double iD = 1.0 / D;
        const double rl[3] = {Sl[0] * iD, Sl[1] * iD, Sl[2] * iD};
        double ru[3];
        lower(gi, rl, ru);                                    // r^i = gamma^ij r_j
        const double sD = 1.0 / sqrt(D);
        const double bu[3] = {Bu[0] * sD, Bu[1] * sD, Bu[2] * sD};
        double bl[3];
        lower(gam, bu, bl);
        Master<MHD> M;
        M.q = tau * iD;
        M.r2 = rl[0] * ru[0] + rl[1] * ru[1] + rl[2] * ru[2];
        M.b2 = bl[0] * bu[0] + bl[1] * bu[1] + bl[2] * bu[2];
        const double rb = rl[0] * bu[0] + rl[1] * bu[1] + rl[2] * bu[2];
        M.rb2 = rb * rb;
        M.gam = a.gm1 + 1.0;
        M.vmax2 = a.vmax2;
        M.prepare();
        // bracket [0, mu+] (g(0) = -1); mu+ is the root itself for cold gas
        // (h = 1), where g(mu+) = 0 up to rounding
        double W = 1.0, eps = 0.0, mu = M.mu_plus(), step, next;
        double lo = 0.0, flo = -1.0, hi = mu, fhi = M.newton(mu, step, next);
        bool ok = fhi >= -1e-12 && M.starts(), done = false;
        if (ok && fhi > 0.0) {
            // Newton steps, held in the bracket by bisections: 2 to 5 on a
            // star; a step of 1e-9 leaves an error at rounding, and where it
            // crossed the end of a clamp (of eps or v) g tells
            for (int it = 0; it < a.max_iter && it < 16; ++it) {
                done = fabs(step) <= a.newton_tol * mu && next > 0.0;
                mu = done || (next > lo && next < hi) ? next : 0.5 * (lo + hi);
                if (done)
                    break;
                const double g = M.newton(mu, step, next);
                if (g < 0.0) {
                    lo = mu;
                    flo = g;
                } else {
                    hi = mu;
                    fhi = g;
                }
            }
        }
        for (bool bracket = ok && fhi > 0.0;; bracket = false) {
            const double g = M.f(mu, W, eps);
            if (!bracket || (done && fabs(g) <= a.g_tol))
                break;
            double Wd, ed;
            auto fm = [&](double m) { return M.f(m, Wd, ed); };
            ok = illinois(fm, lo, hi, flo, fhi, a.tol, a.max_iter, mu);
        }
        if (!ok) {
            st = 3;
        } else {
            const double xx = M.x(mu);
            const double s = mu * xx;
            ut[0] = W * s * (ru[0] + mu * rb * bu[0]);
            ut[1] = W * s * (ru[1] + mu * rb * bu[1]);
            ut[2] = W * s * (ru[2] + mu * rb * bu[2]);
            rho = D / W;
            pr = a.gm1 * rho * eps;
            if (mu * mu * M.rbar2(mu) >= a.vmax2 || W * W - 1.0 > a.ut_max2)
                st = 2;
            else if (!(rho >= a.rho_thr))
                st = 1;
        }
    }
    double *w = a.prim + B.cp_offset + p;
    if (st != 0) {
        rho = a.rho_atm;
        pr = a.p_atm;
        ut[0] = ut[1] = ut[2] = 0.0;
        double q[8];
        p2c_point<MHD>(gam, sg, a.gm1, rho, ut, pr, Bu, q);
#pragma unroll
        for (int i = 0; i < 5; ++i)
            c[i * fs] = q[i];
    }
    w[0] = rho;
    w[fs] = ut[0];
    w[2 * fs] = ut[1];
    w[3 * fs] = ut[2];
    w[4 * fs] = pr;
    if constexpr (MHD) {
        w[5 * fs] = Bu[0];
        w[6 * fs] = Bu[1];
        w[7 * fs] = Bu[2];
    }
    if (a.status)
        a.status[B.cf_offset + p] = st;
}

int share(int n, int most)
{
    const int parts = (n + most - 1) / most;
    return (n + parts - 1) / parts;
}

// Extents w x h of the columns over nx x ny outputs (rows stored `row` apart):
// the widest a workgroup can hold, unless a narrower one needs a quarter fewer
// (wide pieces of rows: the 7 metric fields of 8 x 128^3 cells 565 us, with the
// fewest columns 660; short of 129 points the fewest are often the widest).
// The even share of the outputs, not full columns and a remainder.
void column_shape(int nx, int ny, int row, int &w, int &h)
{
    long long best = INT64_MAX;
    w = h = 1;
    for (int a = std::min(nx, 64); a >= 1; --a) {
        // at order 6: a thread per output, a thread per two points of an input
        // plane (rows of even length), a thread per pair of x sums; offsets below
        // OUTSIDE
        const int b = std::min({ny, INT_ / a, 2 * INT_ / ((a + 6) & ~1) - 5,
                                INT_ / ((a + 1) / 2) - 5,
                                std::max(1, (int)((OUTSIDE / 8 - 64) / row))});
        if (b < 1)
            continue;
        const long long c = ((nx + a - 1LL) / a) * ((ny + b - 1LL) / b);
        if (best == INT64_MAX || 4 * c < 3 * best) {
            best = c;
            w = a;
            h = b;
        }
    }
    w = share(nx, w);
    h = share(ny, h);
}

// Cuts nx x ny x nz outputs of a block into columns of up to `most` planes.
void cut_columns(int block, int nx, int ny, int nz, int row, int most, std::vector<ITile> &out)
{
    int w, h;
    column_shape(nx, ny, row, w, h);
    const int d = share(nz, most);
    for (int k = 0; k < nz; k += d)
        for (int j = 0; j < ny; j += h)
            for (int i = 0; i < nx; i += w)
                out.push_back({block, i, j, k, w, h, d});
}

template <bool TO_CC>
hipError_t launch_interp(int order, const z4c_mplan *P, int ext, const double *in, double *out,
                         hipStream_t s)
{
    const ITile *tiles = (const ITile *)(TO_CC ? P->cc_tiles_d : P->vc_tiles_d);
    const int n = TO_CC ? P->n_cc : P->n_vc, fields = TO_CC ? 7 : 10;
    if (n == 0)
        return hipSuccess;
    // a workgroup per column and field where a grid, which holds less than 2^32
    // threads, can hold them, else as few fields in turn as it takes
    int nf = 1;
    while (nf < fields && (long long)n * ((fields + nf - 1) / nf) > UINT32_MAX / INT_)
        ++nf;
    const int grid = n * ((fields + nf - 1) / nf);
    if (order == 2)
        interp_kernel<2, TO_CC><<<grid, INT_, 0, s>>>(P->blocks_d, tiles, n, nf, ext, in, out);
    else if (order == 4)
        interp_kernel<4, TO_CC><<<grid, INT_, 0, s>>>(P->blocks_d, tiles, n, nf, ext, in, out);
    else
        interp_kernel<6, TO_CC><<<grid, INT_, 0, s>>>(P->blocks_d, tiles, n, nf, ext, in, out);
    return hipGetLastError();
}

bool aligned8(const void *p) { return ((uintptr_t)p & 7u) == 0; }

z4c_status check_plan(const z4c_mplan *P)
{
    if (!P)
        return set_error(Z4C_EINVAL, "mplan is NULL");
    if (!P->device)
        return set_error(Z4C_ENODEV, "mplan was created without a device");
    return Z4C_OK;
}

z4c_status check_order(int order)
{
    if (order != 2 && order != 4 && order != 6)
        return set_error(Z4C_EINVAL, "interpolation order must be 2, 4 or 6");
    return Z4C_OK;
}

}  // namespace
}  // namespace z4c

using namespace z4c;

extern "C" {

z4c_status z4c_mplan_create(const z4c_mblock *blocks, int nblocks, int flags, z4c_mplan **out)
{
    if (!out)
        return set_error(Z4C_EINVAL, "out is NULL");
    *out = nullptr;
    if (!blocks || nblocks < 1)
        return set_error(Z4C_EINVAL, "blocks is NULL or nblocks < 1");
    if (flags & ~Z4C_PLAN_NO_DEVICE)
        return set_error(Z4C_EINVAL, "unknown flags");
    std::vector<ITile> cc, vc;
    std::vector<MTile> pt;
    long long columns = 0;
    for (int b = 0; b < nblocks; ++b) {
        const z4c_mblock &B = blocks[b];
        char buf[160];
        if (B.ncx < 1 || B.ncy < 1 || B.ncz < 1 || B.ngv < 0 || B.ngc < 0) {
            snprintf(buf, sizeof buf, "block %d: cells must be >= 1 and ghosts >= 0", b);
            return set_error(Z4C_EINVAL, buf);
        }
        if (B.vs_offset < 0 || B.vm_offset < 0 || B.cg_offset < 0 || B.cp_offset < 0
            || B.ca_offset < 0 || B.cq_offset < 0 || B.cf_offset < 0 || B.vc_stride < 0
            || B.cc_stride < 0) {
            snprintf(buf, sizeof buf, "block %d: offsets and strides must be >= 0", b);
            return set_error(Z4C_EINVAL, buf);
        }
        const long long nv = (long long)(B.ncx + 1 + 2 * B.ngv) * (B.ncy + 1 + 2 * B.ngv)
                           * (B.ncz + 1 + 2 * B.ngv);
        const long long nc = (long long)(B.ncx + 2 * B.ngc) * (B.ncy + 2 * B.ngc)
                           * (B.ncz + 2 * B.ngc);
        if (B.vc_stride < nv || B.cc_stride < nc) {
            snprintf(buf, sizeof buf, "block %d: a field stride is smaller than the stored field", b);
            return set_error(Z4C_EINVAL, buf);
        }
        const int sc[3] = {B.ncx + 2 * B.ngc, B.ncy + 2 * B.ngc, B.ncz + 2 * B.ngc};
        const long long ncs = (long long)sc[0] * sc[1] * sc[2];
        if (ncs > INT32_MAX) {
            snprintf(buf, sizeof buf, "block %d: more than 2^31 stored cells", b);
            return set_error(Z4C_EINVAL, buf);
        }
        for (long long c = 0; c < ncs; c += PNT)
            pt.push_back({b, (int)c});
        int w, h;
        column_shape(sc[0], sc[1], sc[0], w, h);
        columns += ((sc[0] + w - 1LL) / w) * ((sc[1] + h - 1LL) / h);
    }
    // Planes of a column: long ones read fewer planes twice, few blocks need
    // short ones to occupy the chip (10 fields, at most 17 / 33 / 65 planes: 1 x
    // 64^3 cells, 22 columns, 16 / 18 / 24 us; 2 x 64^3 26 / 23 / 29 us; 1 x
    // 128^3, 80 columns, 119 / 109 / 106 us; 8 x 128^3 887 / 807 / 783 us).
    const int most = (int)std::min(std::max(columns, 17LL), 65LL);
    for (int b = 0; b < nblocks; ++b) {
        const z4c_mblock &B = blocks[b];
        const int gc = 2 * B.ngc;
        cut_columns(b, B.ncx + gc, B.ncy + gc, B.ncz + gc, B.ncx + gc, most, cc);
        cut_columns(b, B.ncx + 1, B.ncy + 1, B.ncz + 1, B.ncx + 1 + 2 * B.ngv, most, vc);
    }
    if (cc.size() > (size_t)INT32_MAX || vc.size() > (size_t)INT32_MAX
        || pt.size() > (size_t)INT32_MAX)
        return set_error(Z4C_EINVAL, "too many tiles");
    z4c_mplan *P = new z4c_mplan;
    P->blocks.assign(blocks, blocks + nblocks);
    P->n_cc = (int)cc.size();
    P->n_vc = (int)vc.size();
    P->n_pt = (int)pt.size();
    if (!(flags & Z4C_PLAN_NO_DEVICE)) {
        hipError_t e = hipMalloc(&P->blocks_d, sizeof(z4c_mblock) * nblocks);
        if (e == hipSuccess)
            e = hipMalloc(&P->cc_tiles_d, sizeof(ITile) * cc.size());
        if (e == hipSuccess)
            e = hipMalloc(&P->vc_tiles_d, sizeof(ITile) * vc.size());
        if (e == hipSuccess)
            e = hipMalloc(&P->pt_tiles_d, sizeof(MTile) * pt.size());
        if (e == hipSuccess)
            e = hipMemcpy(P->blocks_d, blocks, sizeof(z4c_mblock) * nblocks,
                          hipMemcpyHostToDevice);
        if (e == hipSuccess)
            e = hipMemcpy(P->cc_tiles_d, cc.data(), sizeof(ITile) * cc.size(),
                          hipMemcpyHostToDevice);
        if (e == hipSuccess)
            e = hipMemcpy(P->vc_tiles_d, vc.data(), sizeof(ITile) * vc.size(),
                          hipMemcpyHostToDevice);
        if (e == hipSuccess)
            e = hipMemcpy(P->pt_tiles_d, pt.data(), sizeof(MTile) * pt.size(),
                          hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            z4c_mplan_destroy(P);
            return e == hipErrorOutOfMemory ? set_error(Z4C_ENOMEM, "hipMalloc(mplan tables)")
                                            : set_hip_error(e, "mplan tables");
        }
        P->device = true;
    }
    *out = P;
    return Z4C_OK;
}

z4c_status z4c_mplan_destroy(z4c_mplan *P)
{
    if (!P)
        return Z4C_OK;
    if (P->blocks_d)
        (void)hipFree(P->blocks_d);
    if (P->cc_tiles_d)
        (void)hipFree(P->cc_tiles_d);
    if (P->vc_tiles_d)
        (void)hipFree(P->vc_tiles_d);
    if (P->pt_tiles_d)
        (void)hipFree(P->pt_tiles_d);
    delete P;
    return Z4C_OK;
}

z4c_status z4c_metric_to_cc(const z4c_mplan *P, int order, int ext, const double *u,
                            double *geom, void *stream)
{
    z4c_status st;
    if (!P)
        return set_error(Z4C_EINVAL, "mplan is NULL");
    if ((st = check_order(order)) != Z4C_OK)
        return st;
    if (!u || !geom)
        return set_error(Z4C_EINVAL, "u and geom must not be NULL");
    if ((const void *)u == (const void *)geom)
        return set_error(Z4C_EINVAL, "geom must not alias u");
    if (!aligned8(u) || !aligned8(geom))
        return set_error(Z4C_EALIGN, "arrays must be 8-byte aligned");
    if (ext < 0)
        return set_error(Z4C_EINVAL, "ext must be >= 0");
    for (size_t b = 0; b < P->blocks.size(); ++b) {
        const z4c_mblock &B = P->blocks[b];
        char buf[160];
        if (ext > B.ngc) {
            snprintf(buf, sizeof buf, "block %zu: ext %d exceeds the %d stored ghost cells", b, ext,
                     B.ngc);
            return set_error(Z4C_EINVAL, buf);
        }
        if (B.ngv < order / 2 - 1 + ext) {
            snprintf(buf, sizeof buf, "block %zu: order %d to %d ghost cells needs %d ghost "
                     "vertices, %d stored", b, order, ext, order / 2 - 1 + ext, B.ngv);
            return set_error(Z4C_ENOGHOST, buf);
        }
    }
    if ((st = check_plan(P)) != Z4C_OK)
        return st;
    const hipError_t e = launch_interp<true>(order, P, ext, u, geom, (hipStream_t)stream);
    return e == hipSuccess ? Z4C_OK : set_hip_error(e, "interpolation kernel launch");
}

z4c_status z4c_sources_to_vc(const z4c_mplan *P, int order, const double *adm, double *matter,
                             void *stream)
{
    z4c_status st;
    if (!P)
        return set_error(Z4C_EINVAL, "mplan is NULL");
    if ((st = check_order(order)) != Z4C_OK)
        return st;
    if (!adm || !matter)
        return set_error(Z4C_EINVAL, "adm and matter must not be NULL");
    if ((const void *)adm == (const void *)matter)
        return set_error(Z4C_EINVAL, "matter must not alias adm");
    if (!aligned8(adm) || !aligned8(matter))
        return set_error(Z4C_EALIGN, "arrays must be 8-byte aligned");
    for (size_t b = 0; b < P->blocks.size(); ++b) {
        const z4c_mblock &B = P->blocks[b];
        if (B.ngc < order / 2) {
            char buf[160];
            snprintf(buf, sizeof buf, "block %zu: order %d needs %d ghost cells, %d stored", b,
                     order, order / 2, B.ngc);
            return set_error(Z4C_ENOGHOST, buf);
        }
    }
    if ((st = check_plan(P)) != Z4C_OK)
        return st;
    const hipError_t e = launch_interp<false>(order, P, 0, adm, matter, (hipStream_t)stream);
    return e == hipSuccess ? Z4C_OK : set_hip_error(e, "interpolation kernel launch");
}

z4c_status z4c_adm_sources(const z4c_mplan *P, const z4c_fluid *fluid, int ext,
                           const double *geom, const double *prim, double *adm, void *stream)
{
    z4c_status st;
    if (!P)
        return set_error(Z4C_EINVAL, "mplan is NULL");
    if (!fluid || !geom || !prim || !adm)
        return set_error(Z4C_EINVAL, "fluid, geom, prim and adm must not be NULL");
    if (fluid->mhd != 0 && fluid->mhd != 1)
        return set_error(Z4C_EINVAL, "mhd must be 0 or 1");
    if (!(fluid->gamma_ad > 1.0) || !std::isfinite(fluid->gamma_ad))
        return set_error(Z4C_EINVAL, "gamma_ad must be finite and > 1");
    if (!(fluid->chi_floor > 0.0) || !std::isfinite(fluid->chi_floor))
        return set_error(Z4C_EINVAL, "chi_floor must be finite and > 0");
    if ((const void *)adm == (const void *)geom || (const void *)adm == (const void *)prim)
        return set_error(Z4C_EINVAL, "adm must not alias geom or prim");
    if (!aligned8(geom) || !aligned8(prim) || !aligned8(adm))
        return set_error(Z4C_EALIGN, "arrays must be 8-byte aligned");
    if (ext < 0)
        return set_error(Z4C_EINVAL, "ext must be >= 0");
    for (size_t b = 0; b < P->blocks.size(); ++b)
        if (ext > P->blocks[b].ngc) {
            char buf[160];
            snprintf(buf, sizeof buf, "block %zu: ext %d exceeds the %d stored ghost cells", b,
                     ext, P->blocks[b].ngc);
            return set_error(Z4C_EINVAL, buf);
        }
    if ((st = check_plan(P)) != Z4C_OK)
        return st;
    if (P->n_pt == 0)
        return Z4C_OK;
    const double gfac = fluid->gamma_ad / (fluid->gamma_ad - 1.0);
    const MTile *tiles = (const MTile *)P->pt_tiles_d;
    if (fluid->mhd)
        adm_kernel<true><<<P->n_pt, PNT, 0, (hipStream_t)stream>>>(
            P->blocks_d, tiles, ext, gfac, fluid->chi_floor, geom, prim, adm);
    else
        adm_kernel<false><<<P->n_pt, PNT, 0, (hipStream_t)stream>>>(
            P->blocks_d, tiles, ext, gfac, fluid->chi_floor, geom, prim, adm);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? Z4C_OK : set_hip_error(e, "ADM source kernel launch");
}

static z4c_status c2p_common(const z4c_mplan *P, const z4c_c2p_params *c, int ext,
                             const void *geom, const void *a, const void *b, C2PArgs &A)
{
    if (!P)
        return set_error(Z4C_EINVAL, "mplan is NULL");
    if (!c || !geom || !a || !b)
        return set_error(Z4C_EINVAL, "params and arrays must not be NULL");
    if (c->mhd != 0 && c->mhd != 1)
        return set_error(Z4C_EINVAL, "mhd must be 0 or 1");
    if (!(c->gamma_ad > 1.0) || !std::isfinite(c->gamma_ad))
        return set_error(Z4C_EINVAL, "gamma_ad must be finite and > 1");
    if (!(c->chi_floor > 0.0) || !std::isfinite(c->chi_floor))
        return set_error(Z4C_EINVAL, "chi_floor must be finite and > 0");
    if (!(c->rho_atm > 0.0) || !(c->p_atm >= 0.0) || !(c->f_thr >= 0.0)
        || !std::isfinite(c->rho_atm) || !std::isfinite(c->p_atm) || !std::isfinite(c->f_thr))
        return set_error(Z4C_EINVAL, "rho_atm > 0, p_atm >= 0 and f_thr >= 0 must be finite");
    if (!(c->ut_max > 0.0) || !std::isfinite(c->ut_max) || !(c->tol > 0.0) || c->max_iter < 1)
        return set_error(Z4C_EINVAL, "ut_max and tol must be > 0, max_iter >= 1");
    if (a == b || a == geom || b == geom)
        return set_error(Z4C_EINVAL, "geom, input and output arrays must not alias");
    if (!aligned8(geom) || !aligned8(a) || !aligned8(b))
        return set_error(Z4C_EALIGN, "arrays must be 8-byte aligned");
    if (ext < 0)
        return set_error(Z4C_EINVAL, "ext must be >= 0");
    for (size_t k = 0; k < P->blocks.size(); ++k)
        if (ext > P->blocks[k].ngc) {
            char buf[160];
            snprintf(buf, sizeof buf, "block %zu: ext %d exceeds the %d stored ghost cells", k,
                     ext, P->blocks[k].ngc);
            return set_error(Z4C_EINVAL, buf);
        }
    z4c_status st = check_plan(P);
    if (st != Z4C_OK)
        return st;
    A = C2PArgs{};
    A.blocks = P->blocks_d;
    A.tiles = (const MTile *)P->pt_tiles_d;
    A.ext = ext;
    A.mhd = c->mhd;
    A.max_iter = c->max_iter;
    A.gm1 = c->gamma_ad - 1.0;
    A.chi_floor = c->chi_floor;
    A.rho_atm = c->rho_atm;
    A.p_atm = c->p_atm;
    A.eps_atm = c->p_atm / ((c->gamma_ad - 1.0) * c->rho_atm);
    A.rho_thr = c->f_thr * c->rho_atm;
    A.ut_max2 = c->ut_max * c->ut_max;
    A.vmax2 = A.ut_max2 / (1.0 + A.ut_max2);
    A.tol = c->tol;
    A.newton_tol = std::max(c->tol, 1e-9);
    A.g_tol = std::max(c->tol, 1e-14);
    A.geom = (const double *)geom;
    return Z4C_OK;
}

z4c_status z4c_p2c(const z4c_mplan *P, const z4c_c2p_params *c, int ext, const double *geom,
                   const double *prim, double *cons, void *stream)
{
    C2PArgs A;
    const z4c_status st = c2p_common(P, c, ext, geom, prim, cons, A);
    if (st != Z4C_OK)
        return st;
    if (P->n_pt == 0)
        return Z4C_OK;
    A.prim_in = prim;
    A.cons = cons;
    if (c->mhd)
        p2c_kernel<true><<<P->n_pt, PNT, 0, (hipStream_t)stream>>>(A);
    else
        p2c_kernel<false><<<P->n_pt, PNT, 0, (hipStream_t)stream>>>(A);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? Z4C_OK : set_hip_error(e, "p2c kernel launch");
}

z4c_status z4c_c2p(const z4c_mplan *P, const z4c_c2p_params *c, int ext, const double *geom,
                   double *cons, double *prim, int *status, void *stream)
{
    C2PArgs A;
    const z4c_status st = c2p_common(P, c, ext, geom, cons, prim, A);
    if (st != Z4C_OK)
        return st;
    if (status && (((uintptr_t)status & 3u) != 0))
        return set_error(Z4C_EALIGN, "status must be 4-byte aligned");
    if (P->n_pt == 0)
        return Z4C_OK;
    A.cons = cons;
    A.prim = prim;
    A.status = status;
    if (c->mhd)
        c2p_kernel<true><<<P->n_pt, PNT, 0, (hipStream_t)stream>>>(A);
    else
        c2p_kernel<false><<<P->n_pt, PNT, 0, (hipStream_t)stream>>>(A);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? Z4C_OK : set_hip_error(e, "c2p kernel launch");
}

}  // extern "C"
