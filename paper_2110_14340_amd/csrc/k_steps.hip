// Several Jacobi sweeps between two arrays in one launch, for gfx950.
//
// A sweep of a small grid in a graph is bound by its launch, a large one by HBM.
// Here a workgroup loads a region of 64 columns and 8 R rows once, advances it
// T steps in registers and stores the cells that are still right, those T or
// more away from the region's sides.  A wave holds R rows, lane = column:
// left and right neighbours come by DPP, the rows above and below it from the
// waves beside it through LDS, one barrier a step.  Neighbouring regions
// overlap by 2 T: at T = 9 a cell is computed 3.2 times with R = 4 and 1.9 times
// with R = 8.  Steps in a graph of 40, us a step, one launch each and here: 64^2
// 3.6 and 1.2, 512^2 over 4 partitions 4.6 and 1.5, 3000x700 over 8 12.7 and 3.5,
// 2048^2 over 2 16.2 and 4.6, 8192^2 over 8 171 and 61 (there 2.2e12 computed
// cells a second).  T = 5 and 7 took 74.6 and 66.8 at 8192^2, 13 with R = 8
// 66.2; R = 12 and 16 128 and 209.
//
// An odd T takes the step from one array to the other, as a single step would:
// a region reads the input array only and writes the output array only, so no
// workgroup waits for another.  Cells outside the box keep what their array
// holds: a step of odd number reads them from the input array, one of even
// number from the output array, and both are loaded.  Every cell's additions
// are those of the single sweep, in the same order.
#include "k_common.h"
#include "kernels.h"

namespace jk {

namespace {

constexpr int kChainWaves = 8;
constexpr int kChainThreads = kChainWaves * kWave;

typedef const __attribute__((address_space(4))) ChainPart ConstChainPart;
typedef const __attribute__((address_space(4))) Chain ConstChain;
typedef __attribute__((address_space(1))) double GDouble;
typedef const __attribute__((address_space(1))) double ConstGDouble;

__device__ __forceinline__ int part_of(ConstChainPart *p, int n, int64_t row, int q) {
    while (q + 1 < n && row >= p[q].hi) ++q;
    return q;
}

template <int R>
__global__ void __launch_bounds__(kChainThreads)
jacobi_chain_kernel(Chain ch, int T, int64_t gx, int64_t tiles) {
    __shared__ double edge_rows[2][kChainWaves][2][kWave];
    const int64_t b = blockIdx.x;
    const int64_t t = (b & 7) * ((int64_t)gridDim.x >> 3) + (b >> 3);  // neighbouring regions on one XCD
    if (t >= tiles) return;  // the whole workgroup
    ConstChain *cc = (ConstChain *)&ch;
    ConstChainPart *part = &cc->p[0];
    const int n = cc->n;
    const int64_t nx = cc->nx, ny = cc->ny, r_lo = cc->lo[0], r_hi = cc->hi[0], c_lo = cc->lo[1], c_hi = cc->hi[1];
    const int lane = threadIdx.x & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t ty = (uint32_t)t / (uint32_t)gx, tx = (uint32_t)t % (uint32_t)gx;
    const int64_t tile_r = r_lo + (int64_t)ty * (kChainWaves * R - 2 * T), tile_c = c_lo + (int64_t)tx * (kWave - 2 * T);
    const int64_t row0 = tile_r - T + (int64_t)w * R, col = tile_c - T + lane;
    const bool in_row = col >= 0 && col < nx, box_col = col >= c_lo && col < c_hi;
    const bool sides = tile_r - T < r_lo || tile_r - T + kChainWaves * R > r_hi || tile_c - T < c_lo ||
                       tile_c - T + kWave > c_hi;
    double v[R], o[R];
    int q = 0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int64_t row = row0 + k;
        v[k] = 0.0;
        o[k] = 0.0;
        if (row < 0 || row >= ny) continue;
        q = part_of(part, n, row, q);
        if (in_row) {
            v[k] = ((ConstGDouble *)part[q].in)[row * nx + col];
            if (sides && !(box_col && row >= r_lo && row < r_hi)) o[k] = ((ConstGDouble *)part[q].out)[row * nx + col];
        }
    }
    auto advance = [&](int s, auto box) {  // box(k): row k of this lane is computed
        edge_rows[s & 1][w][0][lane] = v[0];
        edge_rows[s & 1][w][1][lane] = v[R - 1];
        __syncthreads();
        const double above = w > 0 ? edge_rows[s & 1][w - 1][1][lane] : 0.0;
        const double below = w < kChainWaves - 1 ? edge_rows[s & 1][w + 1][0][lane] : 0.0;
        double prev = above;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const double mid = v[k], next = k + 1 < R ? v[k + 1] : below;
            const double vert = prev + next;
            const double horz = dpp<0x138>(mid) + dpp<0x130>(mid);  // wave_shr 1, wave_shl 1: left, right
            box(k, 0.25 * (vert + horz));
            prev = mid;
        }
    };
    if (sides) {
        for (int s = 0; s < T; ++s)
            advance(s, [&](int k, double r) {
                const int64_t row = row0 + k;
                const double mid = v[k];
                v[k] = box_col && row >= r_lo && row < r_hi ? r : o[k];
                o[k] = mid;
            });
    } else {
        for (int s = 0; s < T; ++s) advance(s, [&](int k, double r) { v[k] = r; });
    }
    if (lane < T || lane >= kWave - T || col >= c_hi) return;
    q = 0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int64_t row = row0 + k;
        if (row < tile_r || row >= tile_r + kChainWaves * R - 2 * T || row >= r_hi) continue;
        q = part_of(part, n, row, q);
        ((GDouble *)part[q].out)[row * nx + col] = v[k];
#pragma unroll
        for (int m = 0; m < 2; ++m)
            if (m < part[q].mir.n && row >= part[q].mir.m[m].lo && row < part[q].mir.m[m].hi)
                ((GDouble *)part[q].mir.m[m].ptr)[row * nx + col] = v[k];
    }
}

template <int R>
int64_t chain_tiles(const Chain &ch, int T, int64_t *gx) {
    const int64_t h = kChainWaves * R - 2 * T, w = kWave - 2 * T;
    *gx = (ch.hi[1] - ch.lo[1] + w - 1) / w;
    return *gx * ((ch.hi[0] - ch.lo[0] + h - 1) / h);
}

}  // namespace

// A region takes its 32 or 64 rows' time whatever the box fills of them, so wide
// boxes of few rows take a launch a step (us a step alone and in chains of 40:
// 1000000 columns, 1 row 7.8 and 29, 6 rows 19 and 30, 12 rows 32 and 31; 200000
// columns, 1 row 3.6 and 6.7, 6 rows 6.8 and 7.2, 12 rows 9.8 and 7.5; 20000
// columns, 1 row 3.1 and 1.5).
bool steps_share(const Chain &ch) { return ch.hi[0] - ch.lo[0] >= 12 || ch.hi[1] - ch.lo[1] < 50000; }

hipError_t launch_steps(const Chain &ch, int steps, hipStream_t s) {
    if (ch.n < 1 || ch.n > kMaxPack || steps < 1 || steps > kChainMax || steps % 2 == 0) return hipErrorInvalidValue;
    if (ch.hi[0] <= ch.lo[0] || ch.hi[1] <= ch.lo[1]) return hipSuccess;
    int64_t gx;
    // regions of 64 rows where they fill the chip, else of 32 (R = 8 and 4, us a
    // step in runs of 40: 512^2 1.57 and 1.38, 850^2 2.05 and 1.95, 1000^2 2.20
    // and 2.38, 2048^2 4.7 and 6.4, 8192^2 60 and 87)
    int64_t tiles = chain_tiles<8>(ch, steps, &gx);
    const bool tall = tiles >= 400;
    if (!tall) tiles = chain_tiles<4>(ch, steps, &gx);
    const int64_t grid = (tiles + 7) / 8 * 8;
    if (grid > (int64_t)INT32_MAX) return hipErrorInvalidValue;
    if (tall)
        hipLaunchKernelGGL(jacobi_chain_kernel<8>, dim3((unsigned)grid), dim3(kChainThreads), 0, s, ch, steps, gx, tiles);
    else
        hipLaunchKernelGGL(jacobi_chain_kernel<4>, dim3((unsigned)grid), dim3(kChainThreads), 0, s, ch, steps, gx, tiles);
    return hipGetLastError();
}

}  // namespace jk
