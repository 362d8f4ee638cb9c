// z4c_kernels.hip -- gfx950 kernels of the Z4c hot path other than the tile
// kernels (those live in z4c_tile.h, instantiated in z4c_variants_*.hip):
// ghost refresh, per-block norm reduction, non-finite scan, and the dispatch
// to the tile-kernel variants.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>
#include <utility>

#include "z4c_internal.h"

namespace z4c {
namespace {

// ---------------------------------------------------------------------------
// Ghost refresh: one thread per ghost point, all 22 fields, every load issued
// before the first store.  What bounds it: memory on large sets, where the
// pieces of 4 points at the ends of rows are parts of sectors that it reads,
// merges and writes back; latency on small ones.  Against a loop that waited
// for each field, 64-bit divisions and one slab per end: 512 blocks of 16^3
// 502 -> 424 us, 8 x 128^3 452 -> 406 us (436 with neighbouring workgroups on
// different XCDs), one of 16^3 8.8 -> 3.9 us.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) ghost_kernel(const GhostArgs g, long long total)
{
    const long long gid = (long long)xcd_logical(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
    if (gid >= total)
        return;
    // block by binary search over the prefix sums
    int lo = 0, hi = g.nblocks;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (g.ghost_start[mid] <= gid)
            lo = mid;
        else
            hi = mid;
    }
    const int b = lo;
    const z4c_block B = g.blocks[b];
    // 32 bits hold the ghost points of a block (22 fields each, in memory)
    unsigned r = (unsigned)(gid - g.ghost_start[b]);
    const int ng = B.ng;
    const unsigned ex = B.nx + 2 * ng, ey = B.ny + 2 * ng;
    int i, j, k;
    // z slabs (full planes), then y slabs (interior z), then the ends of the rows
    const unsigned zslab = ng * ey * ex, yslab = ng * B.nz * ex;
    if (r < 2 * zslab) {
        const int side = r >= zslab;
        r -= side * zslab;
        const unsigned row = r / ex, kk = row / ey;
        k = side ? B.nz + (int)kk : (int)kk - ng;
        j = (int)(row - kk * ey) - ng;
        i = (int)(r - row * ex) - ng;
    } else if ((r -= 2 * zslab) < 2 * yslab) {
        const int side = r >= yslab;
        r -= side * yslab;
        const unsigned row = r / ex, kk = row / ng, jj = row - kk * ng;
        k = (int)kk;
        j = side ? B.ny + (int)jj : (int)jj - ng;
        i = (int)(r - row * ex) - ng;
    } else {
        // both ends of a row: the upper one and the next row's lower one are
        // neighbours in memory
        r -= 2 * yslab;
        const unsigned row = r / (2 * ng), ii = r - row * 2 * ng;
        k = (int)(row / B.ny);
        j = (int)(row - k * B.ny);
        i = ii < (unsigned)ng ? (int)ii - ng : B.nx + (int)ii - ng;
    }
    const int ox = i < 0 ? -1 : (i >= B.nx ? 1 : 0);
    const int oy = j < 0 ? -1 : (j >= B.ny ? 1 : 0);
    const int oz = k < 0 ? -1 : (k >= B.nz ? 1 : 0);
    const long long dst = (long long)(k + ng) * ey * ex + (long long)(j + ng) * ex + (i + ng);
    int src_b = -1;
    if (g.policy == Z4C_GHOST_PERIODIC)
        src_b = b;
    else if (g.policy == Z4C_GHOST_NEIGHBOUR)
        src_b = g.neighbours[b * 27 + (oz + 1) * 9 + (oy + 1) * 3 + (ox + 1)];
    const double *src;
    long long sfs = B.field_stride;
    if (src_b < 0) {
        if (!g.frozen)
            return;
        src = g.frozen + B.offset + dst;
    } else {
        const z4c_block Sb = g.blocks[src_b];
        const int si = i - ox * B.nx, sj = j - oy * B.ny, sk = k - oz * B.nz;
        const int sex = Sb.nx + 2 * Sb.ng, sey = Sb.ny + 2 * Sb.ng;
        src = g.u + Sb.offset + (long long)(sk + Sb.ng) * sey * sex
            + (long long)(sj + Sb.ng) * sex + (si + Sb.ng);
        sfs = Sb.field_stride;
    }
    double *out = g.u + B.offset + dst;
    double v[NFIELD];
#pragma unroll
    for (int f = 0; f < NFIELD; ++f)
        v[f] = src[f * sfs];
#pragma unroll
    for (int f = 0; f < NFIELD; ++f)
        out[f * B.field_stride] = v[f];
}

// Per-block norms from per-tile partial sums, a workgroup per block: thread
// (g, q) sums norm q over the tiles g, g + NORM_GROUPS, ..., then the groups'
// sums meet by halves; the order depends on the tile count alone.  Latency bounds it
// (a few loads per thread): with one thread per norm 8 blocks of 250 tiles
// took 88 us, now 6.
constexpr int NORM_THREADS = 1024, NORM_GROUPS = NORM_THREADS / 16;

__global__ void __launch_bounds__(NORM_THREADS)
norm_reduce_kernel(const z4c_block *blocks, int nblocks, const long long *tile_start,
                   const int *tile_count, const double *partial, double *norms)
{
    __shared__ double sum[NORM_THREADS];
    const int t = threadIdx.x;
    for (int b = blockIdx.x; b < nblocks; b += gridDim.x) {
        const double *p = partial + tile_start[b] * 16 + t % 16;
        const int n = tile_count[b];
        double s = 0.0;
#pragma unroll 4
        for (int k = t / 16; k < n; k += NORM_GROUPS)
            s += p[k * 16LL];
        sum[t] = s;
        __syncthreads();
        for (int h = NORM_THREADS / 2; h >= 16; h >>= 1) {
            if (t < h)
                sum[t] += sum[t + h];
            __syncthreads();
        }
        if (t < 16) {
            const z4c_block B = blocks[b];
            norms[b * 16LL + t] = sum[t] * (B.dx * B.dy * B.dz);
        }
        __syncthreads();   // before the next block's sums
    }
}

__global__ void finite_count_kernel(const z4c_block *blocks, int nblocks, const long long *pt_start,
                                    long long total, const double *u, unsigned long long *count)
{
    const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned long long bad = 0;
    if (gid < total) {
        int lo = 0, hi = nblocks;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (pt_start[mid] <= gid)
                lo = mid;
            else
                hi = mid;
        }
        const z4c_block B = blocks[lo];
        const long long r = gid - pt_start[lo];
        const int i = (int)(r % B.nx), j = (int)((r / B.nx) % B.ny), k = (int)(r / ((long long)B.nx * B.ny));
        const int ex = B.nx + 2 * B.ng, ey = B.ny + 2 * B.ng;
        const long long pt = (long long)(k + B.ng) * ey * ex + (long long)(j + B.ng) * ex + (i + B.ng);
        for (int f = 0; f < NFIELD; ++f) {
            const double v = u[B.offset + f * B.field_stride + pt];
            bad += isfinite(v) ? 0ull : 1ull;
        }
    }
    // wave-level sum, one atomic per wave
    for (int off = 32; off >= 1; off >>= 1)
        bad += __shfl_xor(bad, off, 64);
    if ((threadIdx.x & 63) == 0 && bad)
        atomicAdd(count, bad);
}

__global__ void zero_u64_kernel(unsigned long long *p) { *p = 0ull; }

}  // namespace

bool stage_shape_supported(int fd_order, int tx, int ty, int tz, int waves)
{
    if (tx == 8 && ty == 4 && tz == 8)
        return waves == 1 && fd_order == 6;
    if (tx != 8 || ty != 8 || (tz != 8 && tz != 4))
        return false;
    return waves == 2 || (waves == 1 && tz == 4 && fd_order == 6);
}

hipError_t launch_stage(int mode, int fd_order, int arith, int advection, const StageArgs &a,
                        hipStream_t s)
{
    if (a.ntiles <= 0)
        return hipSuccess;
    if (mode == MODE_RK_MON)
        return launch_monitor(fd_order, a, s);
    if (mode != MODE_CONS && advection == Z4C_ADVECT_LOPSIDED)
        return launch_lopsided(mode, fd_order, a, s);
    if (arith == Z4C_ARITH_FP32_NAIVE && mode != MODE_CONS)
        return mode == MODE_RHS ? launch_naive(a, s) : hipErrorInvalidValue;
    if (fd_order == 4)
        return launch_p4(mode, arith, a, s);
    if (mode == MODE_CONS || arith != Z4C_ARITH_FP32)
        return launch_p6_f64(mode, a, s);
    return launch_p6_f32(mode, a, s);
}

hipError_t launch_ghost(const GhostArgs &g, long long total_ghost, hipStream_t s)
{
    if (total_ghost <= 0)
        return hipSuccess;
    const long long nb = (total_ghost + 255) / 256;
    ghost_kernel<<<dim3((unsigned)nb), dim3(256), 0, s>>>(g, total_ghost);
    return hipGetLastError();
}

hipError_t launch_norm_reduce(const z4c_block *blocks, int nblocks, const long long *tile_start,
                              const int *tile_count, const double *partial, double *norms,
                              hipStream_t s)
{
    // a launch holds less than 2^32 threads; more blocks take turns
    const unsigned grid = std::min((unsigned)nblocks, UINT32_MAX / NORM_THREADS);
    norm_reduce_kernel<<<dim3(grid), dim3(NORM_THREADS), 0, s>>>(blocks, nblocks, tile_start,
                                                                 tile_count, partial, norms);
    return hipGetLastError();
}

hipError_t launch_finite_count(const z4c_block *blocks, int nblocks, const long long *pt_start,
                               long long total_pts, const double *u, unsigned long long *count,
                               hipStream_t s)
{
    if (total_pts <= 0)
        return hipSuccess;
    const long long nb = (total_pts + 255) / 256;
    finite_count_kernel<<<dim3((unsigned)nb), dim3(256), 0, s>>>(blocks, nblocks, pt_start,
                                                                total_pts, u, count);
    return hipGetLastError();
}

hipError_t launch_zero_u64(unsigned long long *p, hipStream_t s)
{
    zero_u64_kernel<<<1, 1, 0, s>>>(p);
    return hipGetLastError();
}

}  // namespace z4c
