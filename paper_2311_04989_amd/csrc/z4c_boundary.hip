// z4c_boundary.hip -- radiative (Sommerfeld) outer boundary of a level set.
//
// The paper states no outer boundary condition for Z4c (its static-star
// test moves the outer boundary further out instead of treating it); this is
// the usual radiative law of moving-puncture codes, taken as a reading.  The
// outer ghost points of a block (those in a direction whose neighbour entry
// is -1) advance, in every Runge-Kutta stage, by
//     d_t u = -(x^a / r) D_a u - (u - u_inf) / r,      r = |x|,
// for each of the 22 fields, u_inf its flat-space value (1 for chi, gt_xx,
// gt_yy, gt_zz and alpha, 0 otherwise), D_a the second-order difference
// along a: centred where the point's index along a lies inside the interior
// range, one-sided towards the interior outside it (it reads only stored
// points; samples at ghost points that have a neighbour are read through
// the neighbour rule when the stage reads its halo that way, so that both
// see the same values).  The stage combination and the enforcement (det gt
// = 1, tr At = 0, floors) are those of the interior points; there is no
// dissipation.  The stage kernel writes interior points and this one the
// outer ghost points, and both read only the stage input, so the two run in
// either order.
#include "z4c_tile.h"

namespace z4c {
namespace {

__device__ __forceinline__ double flat_value(int f)
{
    return (f == CHI || f == GXX || f == GYY || f == GZZ || f == ALPHA) ? 1.0 : 0.0;
}

// The fields of an outer point in two parts: the conformal metric and At, which
// the enforcement couples, and the others.
constexpr int NPART[2] = {12, 10};
constexpr int PART[2][12] = {{GXX, GXX + 1, GXX + 2, GXX + 3, GXX + 4, GXX + 5, AXX, AXX + 1, AXX + 2,
                              AXX + 3, AXX + 4, AXX + 5},
                             {CHI, KHAT, THETA, GAMX, GAMX + 1, GAMX + 2, ALPHA, BETAX, BETAX + 1,
                              BETAX + 2}};

constexpr int RAD_THREADS = 256;
constexpr int RAD_AHEAD = 2;   // fields in flight per point

// Advances the fields of part K of one outer point (e0: element offset of field
// 0; smp, A, Q, out: its samples and their use, below).  No read takes a branch
// (a register that the stage does not read is replaced by the centre), so that a
// field's wait leaves the younger reads in flight.
template <bool RHS, int K>
__device__ __forceinline__ void radiative_fields(const RadiativeArgs &a, long long e0, long long fs,
                                                 const double *const (&smp)[3][2],
                                                 const double (&A)[3], const double (&Q)[3],
                                                 const bool (&out)[3], double r)
{
    constexpr int N = NPART[K];
    struct Reads {
        double c, s[3][2], u1, u2;
    };
    const double *uc = a.u + e0, *u1 = a.read_u1 ? a.u1 + e0 : uc, *u2 = a.use_u2 ? a.u2 + e0 : uc;
    auto read = [&](int f) __attribute__((always_inline)) {
        const long long fo = f * fs;
        Reads v;
        v.c = uc[fo];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            v.s[d][0] = smp[d][0][fo];
            v.s[d][1] = smp[d][1][fo];
        }
        v.u1 = RHS ? 0.0 : u1[fo];
        v.u2 = RHS ? 0.0 : u2[fo];
        return v;
    };
    Reads ring[RAD_AHEAD];
#pragma unroll
    for (int m = 0; m < RAD_AHEAD; ++m)
        ring[m] = read(PART[K][m]);
    double w[NFIELD] = {};
#pragma unroll
    for (int m = 0; m < N; ++m) {
        const int f = PART[K][m];
        const Reads v = ring[m % RAD_AHEAD];
        if (m + RAD_AHEAD < N)
            ring[m % RAD_AHEAD] = read(PART[K][m + RAD_AHEAD]);
        double adv = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double b = out[d] ? v.c : 0.0;
            const double s1 = A[d] * (v.s[d][0] - b), s2 = v.s[d][1] - b;
            adv += Q[d] * (A[d] == 4.0 ? s1 - s2 : s1 + s2);
        }
        const double kf = -(adv + (v.c - flat_value(f))) / r;
        const long long e = e0 + f * fs;
        if constexpr (RHS) {
            a.rhs[e] = kf;
        } else {
            const double n1 = (a.read_u1 ? v.u1 : 0.0) + a.delta * v.c + a.eps_dt * kf;
            double s = a.g1 * v.c + a.g2 * n1;
            if (a.use_u2)
                s += a.g3 * v.u2;
            s += a.beta_dt * kf;
            if (a.write_u1)
                a.u1[e] = n1;
            if (f == CHI)
                s = s > a.chi_floor ? s : a.chi_floor;
            if (f == ALPHA)
                s = s > a.alpha_floor ? s : a.alpha_floor;
            if (K == 0)
                w[f] = s;
            else
                a.out[e] = s;
        }
    }
    if constexpr (!RHS && K == 0) {
        tile::enforce(w, a.chi_floor, a.alpha_floor);
#pragma unroll
        for (int m = 0; m < N; ++m)
            a.out[e0 + PART[K][m] * fs] = w[PART[K][m]];
    }
}

// One thread per outer point and part: it finds its samples once and takes the
// fields in turn, the reads of the next RAD_AHEAD in flight.
// What bounds it: memory latency (169,000 points of 8 x 40^3 would be 5 waves per
// SIMD; the 168 registers of the stage mode, twelve held results and two fields in
// flight, leave 3) and the partial sectors of its pieces of 4 points.  Against a workgroup
// of a thread per (field, point), 32 points at a time, whose first 32 threads
// found the samples and enforced while the others waited: 113 -> 78 us per stage
// of 8 x 40^3, 42 -> 15 of 8 x 24^3; with all 22 fields in one thread 81 and 19.
template <bool RHS>
__global__ void __launch_bounds__(RAD_THREADS) radiative_kernel(const RadiativeArgs a)
{
    const unsigned wg = xcd_logical(blockIdx.x, gridDim.x), part = wg & 1;
    const long long first = (long long)(wg >> 1) * RAD_THREADS;
    const long long gid = first + threadIdx.x;
    if (gid >= a.total)
        return;
    // region of the workgroup's first point by binary search over the prefix
    // sums, then of this thread's (a region has at least ng points: the walk is
    // a few steps)
    int lo = 0, hi = a.nregions;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (a.start[mid] <= first)
            lo = mid;
        else
            hi = mid;
    }
    while (lo + 1 < a.nregions && a.start[lo + 1] <= gid)
        ++lo;
    const OuterRegion R = a.regions[lo];
    const z4c_block B = a.blocks[R.block];
    // 32 bits hold the points of a region (22 fields each, in memory)
    const unsigned q = (unsigned)(gid - a.start[lo]), row = q / (unsigned)R.n[0],
                   pl = row / (unsigned)R.n[1];
    const int p[3] = {R.lo[0] + (int)(q - row * R.n[0]), R.lo[1] + (int)(row - pl * R.n[1]),
                      R.lo[2] + (int)pl};
    const int n[3] = {B.nx, B.ny, B.nz}, ng = B.ng;
    const long long sy = B.nx + 2 * ng, sz = sy * (B.ny + 2 * ng), fs = B.field_stride;
    // Element offset (field 0) of stored point (ii, jj, kk) of this block,
    // or, under the neighbour rule, of the point a neighbour copy would
    // bring there (neighbours share nx, ny, nz, ng and the field stride).
    auto locate = [&](int ii, int jj, int kk) __attribute__((always_inline)) {
        long long base = B.offset;
        if (a.nbr) {
            const int ox = ii < 0 ? -1 : (ii >= B.nx ? 1 : 0);
            const int oy = jj < 0 ? -1 : (jj >= B.ny ? 1 : 0);
            const int oz = kk < 0 ? -1 : (kk >= B.nz ? 1 : 0);
            if (ox | oy | oz) {
                const int sb = a.nbr[R.block * 27 + (oz + 1) * 9 + (oy + 1) * 3 + (ox + 1)];
                if (sb >= 0) {
                    base = a.blocks[sb].offset;
                    ii -= ox * B.nx;
                    jj -= oy * B.ny;
                    kk -= oz * B.nz;
                }
            }
        }
        return base + (long long)(kk + ng) * sz + (long long)(jj + ng) * sy + (ii + ng);
    };
    const long long e0 = B.offset + (long long)(p[2] + ng) * sz + (long long)(p[1] + ng) * sy
                       + (p[0] + ng);
    // Second-order difference per direction from two samples: the next two
    // towards the interior outside the interior range, in differences from the
    // centre, +-4 (s1 - c) -+ (s2 - c); else s2 - s1 of the neighbours at -1
    // and +1.  2 h of it goes into Q = x / (2 h).
    const double *smp[3][2];
    double A[3], Q[3];
    bool out[3];
    const double h[3] = {B.dx, B.dy, B.dz};
    double r2 = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const bool below = p[d] < 0, above = p[d] >= n[d];
        out[d] = below || above;
        A[d] = below ? 4.0 : (above ? -4.0 : -1.0);
        int p1[3] = {p[0], p[1], p[2]}, p2[3] = {p[0], p[1], p[2]};
        p1[d] += below ? 1 : -1;
        p2[d] += below ? 2 : (above ? -2 : 1);
        smp[d][0] = a.u + locate(p1[0], p1[1], p1[2]);
        smp[d][1] = a.u + locate(p2[0], p2[1], p2[2]);
        const double x = a.origins[3 * R.block + d] + p[d] * h[d];
        Q[d] = x / (2.0 * h[d]);
        r2 += x * x;
    }
    const double r = sqrt(r2);

    if (part == 0)   // uniform
        radiative_fields<RHS, 0>(a, e0, fs, smp, A, Q, out, r);
    else
        radiative_fields<RHS, 1>(a, e0, fs, smp, A, Q, out, r);
}

}  // namespace

hipError_t launch_radiative(const RadiativeArgs &a, hipStream_t s)
{
    if (a.total <= 0)
        return hipSuccess;
    const long long nb = 2 * ((a.total + RAD_THREADS - 1) / RAD_THREADS);
    if (a.rhs)
        radiative_kernel<true><<<dim3((unsigned)nb), dim3(RAD_THREADS), 0, s>>>(a);
    else
        radiative_kernel<false><<<dim3((unsigned)nb), dim3(RAD_THREADS), 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace z4c
