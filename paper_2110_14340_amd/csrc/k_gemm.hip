// Dense FP64 contraction C = A*B on the gfx950 matrix cores
// (v_mfma_f64_16x16x4f64).
//
// What bounds it: the matrix cores.  One instruction keeps a SIMD's matrix
// core busy for 64 cycles, so a wave that owns 64x64 elements of C needs
// only 8 KB of A and B for 2048 cycles of it, which the vector L1 delivers
// several times over.  Each wave therefore loads its operands straight into
// registers, in the instruction's own layout, a few stages ahead, and runs
// to the end without LDS or barriers.  (Staged through LDS with a barrier a
// 16-deep slab the matrix cores idled 21 % of the time, and rows of odd length
// went through guarded single loads.)  4096^3: 2165 us before, 1865 now, 73.7
// TFLOP/s; 1000x777x1531 308 and 53 us, over 3 partitions 387 and 65 us.
//
// Layout of v_mfma_f64_16x16x4f64, lane l = 16q + c: A operand A[c][q], B
// operand B[q][c], accumulator element r = D[4r + q][c].  Which k a slot q
// stands for, and which column a slot c, is free as long as both operands
// and the write-back agree.  A stage is 8 consecutive k's: slot q of its
// first instruction is k = 2q, of its second k = 2q + 1, and slot c of column
// blocks 2g and 2g+1 are the columns 32g + 2c and 32g + 2c + 1, so each lane's
// operands are pairs of neighbours, loaded 16 bytes at a time.  The k's of a
// row are walked in increasing stages whatever the tile, with no split of
// the k dimension: an element's sum has the same order, and the same bits,
// for every partition count, tile and bounds.
#include "k_common.h"
#include "kernels.h"

namespace jk {

namespace {

constexpr int kGemmThreads = 256;  // 2 x 2 waves
constexpr int kStage = 8;          // k's of a stage

typedef double d4 __attribute__((ext_vector_type(4)));

// Tile of workgroup b: the 8 XCDs take consecutive workgroup ids in turn, so
// XCD x is given the x-th contiguous eighth of the tiles; inside it, tiles
// are walked in groups of 8 tile-rows (column by column), so the
// workgroups resident on one XCD share few A row-panels and B column-panels
// and most panel reads hit that XCD's L2.
// The grid is a multiple of 8; false: a workgroup past the last tile.
__device__ __forceinline__ bool gemm_tile(int64_t tiles_m, int64_t tiles_n, int64_t *ti, int64_t *tj) {
    const int64_t b = blockIdx.x;
    const int64_t t = (b & 7) * (gridDim.x >> 3) + (b >> 3);
    if (t >= tiles_m * tiles_n) return false;
    constexpr int64_t G = 8;
    const int64_t group = t / (G * tiles_n);
    const int64_t first = group * G;
    const int64_t rows = tiles_m - first < G ? tiles_m - first : G;
    const int64_t in_group = t - group * G * tiles_n;
    *ti = first + in_group % rows;
    *tj = in_group / rows;
    return true;
}

// A wave owns MI x NJ blocks of 16 x 16, a workgroup 2 x 2 waves; S stages of
// operands are held, so a stage's loads have S - 1 stages of matrix
// instructions to arrive.  Rows past m_hi are clamped to the last row, column
// pairs past the last to the last pair: in bounds, computed like any other
// and then not stored (or, for the columns of a clamped pair inside the box,
// stored twice with the same bits).  PAIR false loads B by single elements
// (rows of one element have no pair); Off is the type of a lane's byte
// offsets from the wave's uniform base addresses.
template <int MI, int NJ, int S, bool PAIR, typename Off>
__global__ void __launch_bounds__(kGemmThreads, 2)
gemm_kernel(const double *__restrict__ A, const double *__restrict__ B, double *__restrict__ C, int64_t m_lo,
            int64_t m_hi, int64_t n_lo, int64_t n_hi, int64_t K, int64_t N, int64_t tiles_m, int64_t tiles_n) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int c = lane & 15, q = lane >> 4;
    int64_t ti, tj;
    if (!gemm_tile(tiles_m, tiles_n, &ti, &tj)) return;
    const int64_t row0 = m_lo + (ti * 2 + (wave >> 1)) * (16 * MI);
    const int64_t col0 = n_lo + (tj * 2 + (wave & 1)) * (16 * NJ);
    if (row0 >= m_hi || col0 >= n_hi) return;  // no barriers: a wave without elements is done

    const char *ap = (const char *)(A + row0 * K);
    const char *bp = (const char *)B;
    Off aoff[MI], boff[NJ / 2];
    int64_t cs[NJ / 2];  // first column of this lane's pair in each 32-column group
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int64_t r = row0 + 16 * i + c < m_hi ? 16 * i + c : m_hi - 1 - row0;
        aoff[i] = (Off)((r * K + 2 * q) * 8);
    }
#pragma unroll
    for (int g = 0; g < NJ / 2; ++g) {
        const int64_t j = col0 + 32 * g + 2 * c;
        cs[g] = PAIR ? (j < N - 1 ? j : N - 2) : j;
        boff[g] = (Off)((2 * q * N + (PAIR ? cs[g] : 0)) * 8);
    }
    // PAIR false: the columns of a lane are clamped one by one
    auto single = [&](int64_t k, int g, int e) {
        const int64_t j = cs[g] + e < N ? cs[g] + e : N - 1;
        return B[k * N + j];
    };

    d4 acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};

    dpair a[S][MI], b[S][2][NJ / 2];
    // A pair at a uniform base plus a lane's offset.  Large tiles keep the
    // compiler from hoisting the offset's widening out of the loop: the load
    // then takes base and offset as they are, and the two registers a load
    // that this saves hold a third stage (4096^3 with three such products
    // running side by side 2020 -> 1920 us; alone 1871 -> 1865).
    auto at = [&](const char *base, Off off) {
        if constexpr (MI * NJ >= 8) asm volatile("" : "+v"(off));
        return *reinterpret_cast<const dpair *>(base + off);
    };
    int64_t next = 0;  // the stage loaded next: ap and bp are its base addresses
    auto load = [&](int s) {
        const char *b1 = bp + 8 * N;
#pragma unroll
        for (int i = 0; i < MI; ++i) a[s][i] = at(ap, aoff[i]);
#pragma unroll
        for (int g = 0; g < NJ / 2; ++g) {
            if constexpr (PAIR) {
                b[s][0][g] = at(bp, boff[g]);
                b[s][1][g] = at(b1, boff[g]);
            } else {
                const int64_t k = next * kStage + 2 * q;
                b[s][0][g] = dpair{single(k, g, 0), single(k, g, 1)};
                b[s][1][g] = dpair{single(k + 1, g, 0), single(k + 1, g, 1)};
            }
        }
        ap += kStage * 8;
        bp += kStage * 8 * N;
        ++next;
        // the loads stay in stage order, so a wait for one stage leaves the
        // later ones in flight (reordered, the loop waited for nearly all)
        __builtin_amdgcn_sched_barrier(0);
    };
    auto compute = [&](int s) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s][i][t], b[s][t][j / 2][j % 2], acc[i][j], 0, 0, 0);
    };
    const int64_t ns = K / kStage;  // full stages
    if (ns >= S) {
#pragma unroll
        for (int s = 0; s < S; ++s) load(s);
        while (next + S <= ns) {
#pragma unroll
            for (int s = 0; s < S; ++s) {
                compute(s);
                load(s);
            }
        }
        const int rest = (int)(ns - next);  // stages of the last, incomplete round
#pragma unroll
        for (int s = 0; s < S; ++s) {
            compute(s);
            if (s < rest) load(s);
        }
#pragma unroll
        for (int s = 0; s < S - 1; ++s)
            if (s < rest) compute(s);
    } else {
        while (next < ns) {
            load(0);
            compute(0);
        }
    }
    if (ns * kStage < K) {  // the last, partial stage: zeros past the last k on both sides
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int64_t k = ns * kStage + 2 * q + t;
            const bool in = k < K;
#pragma unroll
            for (int i = 0; i < MI; ++i)
                a[0][i][t] = in ? *reinterpret_cast<const double *>(ap + aoff[i] + 8 * t) : 0.0;
#pragma unroll
            for (int g = 0; g < NJ / 2; ++g) {
                b[0][t][g] = dpair{0.0, 0.0};
                if (in) {
                    b[0][t][g].x = single(k, g, 0);
                    b[0][t][g].y = single(k, g, 1);
                }
            }
        }
        compute(0);
    }
    // acc[i][2g + e][r] is C[row0 + 16i + 4r + q][cs[g] + e]
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t gi = row0 + 16 * i + 4 * r + q;
            if (gi >= m_hi) continue;
#pragma unroll
            for (int g = 0; g < NJ / 2; ++g) {
                double *p = C + gi * N + cs[g];
                const double x = acc[i][2 * g][r], y = acc[i][2 * g + 1][r];
                if (cs[g] >= n_lo && cs[g] + 1 < n_hi) {
                    *reinterpret_cast<dpair *>(p) = dpair{x, y};
                } else {  // a pair across the box's edge
                    if (cs[g] >= n_lo && cs[g] < n_hi) p[0] = x;
                    if (cs[g] + 1 >= n_lo && cs[g] + 1 < n_hi) p[1] = y;
                }
            }
        }
}

}  // namespace

namespace {

// Workgroups that end up on one compute unit: a launch deals its workgroups
// to the 32 shader engines (8 XCDs of 4, 8 units each) in turn, starting at
// the same one, and the launches of all partitions run side by side.
int64_t rounds_of(int64_t parts, int64_t wgs) { return (parts * ((wgs + 31) / 32) + 7) / 8; }

// Cycles of matrix instructions a stage costs the busiest compute unit, for
// waves of `blocks` 16x16 blocks: a workgroup puts one wave on each of the
// unit's four SIMDs, 128 cycles a block and stage.  A unit's only workgroup
// also exposes about 55 cycles a stage (measured: 0.14 us a stage with 2
// blocks, 0.26 with 4, 0.93 with 16); several workgroups hide them in each
// other, but the smaller the wave's tile, the more operand bytes a matrix
// instruction needs: `more` is the time of a 4096^3 product against the
// 64x64 tile's (2039 us; 2109 / 2424 / 2854 us for 8 / 4 / 2 blocks).
double stage_cost(int64_t parts, int64_t wgs, int blocks, double more) {
    const int64_t rounds = rounds_of(parts, wgs);
    return rounds == 1 ? 128.0 * blocks + 55.0 : 128.0 * blocks * (double)rounds * more;
}

// Bytes of (unused) LDS a workgroup asks for, so that a compute unit takes no
// more workgroups than its share: the launches of several partitions
// otherwise pile up on some units while others stay idle (4 partitions of
// 256x1024x1024: 77 us without, 48 us with; 3 of 333x777x1531: 112 and 84).
size_t spread_lds(int64_t parts, int64_t wgs) {
    const int64_t rounds = rounds_of(parts, wgs);
    return parts > 1 && rounds <= 3 ? (size_t)(160 * 1024 / (rounds + 1) + 1280) : 0;
}

}  // namespace

hipError_t launch_gemm(const Launch &L, hipStream_t s) {
    // arguments: A (M x K), B (K x N), C (M x N); iteration box rows
    // [lo0, hi0) of C, columns [lo1, hi1)
    const int64_t m = L.hi[0] - L.lo[0], n = L.hi[1] - L.lo[1];
    if (m <= 0 || n <= 0) return hipSuccess;
    const int64_t K = L.a[0].row_elems, N = L.a[2].row_elems;
    auto tiles = [](int64_t e, int blocks) { return (e + 32 * blocks - 1) / (32 * blocks); };
    // more of the smallest tiles than a launch has room for (2^29 rows of one
    // column): the rows in two launches
    if (tiles(m, 1) * tiles(n, 2) > max_groups(kGemmThreads) - 7) {
        if (m <= 32) return hipErrorInvalidValue;
        Launch half = L;
        half.hi[0] = L.lo[0] + (m / 2 + 31) / 32 * 32;  // less than m
        const hipError_t e = launch_gemm(half, s);
        if (e != hipSuccess) return e;
        half.lo[0] = half.hi[0];
        half.hi[0] = L.hi[0];
        return launch_gemm(half, s);
    }
    const int64_t parts = L.beside > 1 ? L.beside : 1;  // launches of the loop running side by side
#define GEMM_LAUNCH(MI, NJ, S, PAIR, OFF)                                                                              \
    do {                                                                                                               \
        const int64_t tm = tiles(m, MI), tn = tiles(n, NJ);                                                            \
        hipLaunchKernelGGL((gemm_kernel<MI, NJ, S, PAIR, OFF>), dim3((unsigned)((tm * tn + 7) / 8 * 8)),               \
                           dim3(kGemmThreads), spread_lds(parts, tm * tn), s, (const double *)L.a[0].ptr, (const double *)L.a[1].ptr,           \
                           (double *)L.a[2].ptr, L.lo[0], L.hi[0], L.lo[1], L.hi[1], K, N, tm, tn);                    \
        return hipGetLastError();                                                                                      \
    } while (0)
    if (N < 2) GEMM_LAUNCH(1, 2, 4, false, int64_t);
    // wave tiles of 64x64, 32x64, 32x32 and 16x32, whichever keeps the
    // busiest compute unit shortest (1024^3: 134 / 77 / 51 / 59 us; 512^3:
    // 71 / 42 / 28 / 21 us; 2048^3: 291 / 304 / 354 / 409 us; 2467x3597x363:
    // 159 / 140 / 138 / 158 us)
    const double c16 = stage_cost(parts, tiles(m, 4) * tiles(n, 4), 16, 1.0);
    const double c8 = stage_cost(parts, tiles(m, 2) * tiles(n, 4), 8, 1.035);
    const double c4 = stage_cost(parts, tiles(m, 2) * tiles(n, 2), 4, 1.19);
    const double c2 = stage_cost(parts, tiles(m, 1) * tiles(n, 2), 2, 1.40);
    const bool big = c16 <= c8 && c16 <= c4 && c16 <= c2, mid = c8 <= c4 && c8 <= c2;
    // 32-bit lane offsets reach 64 rows of A and 8 rows of B.  Beyond, the large
    // tiles take 64-bit ones and a stage less (256 x 2^25, 8 deep: 11.0 ms, 18.5
    // as 16x32 tiles of single loads; 100 x 2^25, 20 deep: 9.0 and 12.3); few
    // rows that are 2^22 long do best with the short stages of the last form
    // (256 x 256, 2^22 deep: 118 ms, 153 in pairs).
    if (K >= ((int64_t)1 << 22) || N >= ((int64_t)1 << 25)) {
        if (big) GEMM_LAUNCH(4, 4, 2, true, int64_t);
        if (mid) GEMM_LAUNCH(2, 4, 3, true, int64_t);
        GEMM_LAUNCH(1, 2, 4, false, int64_t);
    }
    if (big) GEMM_LAUNCH(4, 4, 3, true, uint32_t);
    if (mid) GEMM_LAUNCH(2, 4, 4, true, uint32_t);
    if (c4 <= c2) GEMM_LAUNCH(2, 2, 4, true, uint32_t);
    GEMM_LAUNCH(1, 2, 6, true, uint32_t);
#undef GEMM_LAUNCH
}

}  // namespace jk
