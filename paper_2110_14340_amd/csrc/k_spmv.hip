// CSR sparse matrix-vector product for gfx950: the plain row-parallel form
// and a binned form for x vectors larger than an XCD's L2.
//
// Plain form: G lanes cooperate on one row (G = 4, 8 or 16, by the mean row
// length): lane g of the group adds val[k]*x[col[k]] for k = row_ptr[i] + g,
// + g + G, ... in increasing k, then the group adds its lanes by a fixed
// butterfly.  col/val reads of a group are contiguous; x is gathered.
#include "k_common.h"
#include "kernels.h"

namespace jk {

namespace {

constexpr int kSpmvThreads = 256;

// Orders a wave's LDS accesses before it and after it.
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Lane g's share of the row [kb, ke): its entries' products added in increasing
// k.  Eight of them are in flight at once, so that a long row is not one load's
// latency after the other.  NT: col and val are read once, so they are loaded
// non-temporally and leave the caches to the gathered x.
template <bool NT>
__device__ __forceinline__ double lane_sum(const int32_t *__restrict__ col, const double *__restrict__ val,
                                           const double *__restrict__ x, int32_t kb, int32_t ke, int g, int G) {
    constexpr int kAhead = 8;
    double s = 0.0;
    int64_t k = (int64_t)kb + g;
    for (; k + (kAhead - 1) * G < ke; k += kAhead * G) {
        int32_t c[kAhead];
        double v[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            c[u] = NT ? __builtin_nontemporal_load(&col[k + u * G]) : col[k + u * G];
            v[u] = NT ? __builtin_nontemporal_load(&val[k + u * G]) : val[k + u * G];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) v[u] *= x[c[u]];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) s += v[u];
    }
    for (; k < ke; k += G) {
        const int32_t c = NT ? __builtin_nontemporal_load(&col[k]) : col[k];
        const double v = NT ? __builtin_nontemporal_load(&val[k]) : val[k];
        s += v * x[c];
    }
    return s;
}

constexpr int kWaveRow = 2048;   // entries beyond which a row may be its wave's work
constexpr int kWaveChunk = 512;  // products of it that the wave has in LDS

// Sum of the row [kb, ke) of this lane's group (none: kb == ke), whole in every
// lane of the group.  Where a wave has one to five rows (20 / G) of more than
// kWaveRow entries, its 64 lanes work out their products, 512 at a time in LDS, and
// G of them add those as the group's own lanes would: 2^18 rows of 3 and one of
// 200,000 took 3.4 ms with a group's own lanes, 2.0 so.
template <int G, bool NT>
__device__ __forceinline__ double row_sum(const int32_t *__restrict__ col, const double *__restrict__ val,
                                          const double *__restrict__ x, int32_t kb, int32_t ke, int g,
                                          double (&sh)[kSpmvThreads / kWave][kWaveChunk]) {
    const int lane = threadIdx.x & (kWave - 1);
    const bool is_long = ke - kb > kWaveRow;
    uint64_t longs = __ballot(is_long && g == 0);
    if (__popcll(longs) > 20 / G) longs = 0;
    double s = 0.0;
    if (!longs || !is_long) s = lane_sum<NT>(col, val, x, kb, ke, g, G);
    double *buf = sh[threadIdx.x / kWave];
    for (; longs; longs &= longs - 1) {
        const int first = __builtin_ctzll(longs);  // the row's first lane
        const int64_t b = __shfl(kb, first, kWave), e = __shfl(ke, first, kWave);
        double t = 0.0;
        for (int64_t k0 = b; k0 < e; k0 += kWaveChunk) {
            double v[kWaveChunk / kWave];
#pragma unroll
            for (int u = 0; u < kWaveChunk / kWave; ++u) {
                const int64_t k = k0 + u * kWave + lane;
                v[u] = k < e ? val[k] * x[col[k]] : 0.0;
            }
            wave_order();  // the adds of the chunk before are done
#pragma unroll
            for (int u = 0; u < kWaveChunk / kWave; ++u) buf[u * kWave + lane] = v[u];
            wave_order();
            const int m = (int)(e - k0 < kWaveChunk ? e - k0 : kWaveChunk);
            if (lane < G)
#pragma unroll 16
                for (int k = lane; k < m; k += G) t += buf[k];
        }
        t = __shfl(t, g, kWave);
        if (lane - g == first) s = t;
    }
    return group_sum<G>(s);
}

// Eight waves a SIMD: the gathers' latency is what the plain form waits for.
template <int G, bool NT>
__global__ void __launch_bounds__(kSpmvThreads, 8)
spmv_kernel(const int32_t *__restrict__ rp, const int32_t *__restrict__ col, const double *__restrict__ val,
            const double *__restrict__ x, double *__restrict__ y, int64_t r_lo, int64_t r_hi) {
    const int64_t t = (int64_t)blockIdx.x * kSpmvThreads + threadIdx.x;
    const int64_t i = r_lo + t / G;
    const int g = threadIdx.x & (G - 1);
    __shared__ double sh[kSpmvThreads / kWave][kWaveChunk];
    const bool live = i < r_hi;
    const double s = row_sum<G, NT>(col, val, x, live ? rp[i] : 0, live ? rp[i + 1] : 0, g, sh);
    if (live && g == 0) y[i] = s;
}

// The partitions of one product in one launch: partition q's rows take the
// workgroups from wg_begin on, each row summed as its own launch would.
struct SpmvPart {
    const int32_t *rp, *col;
    const double *val, *x;
    double *y;
    int64_t lo, hi, wg_begin;
};
struct SpmvParts {
    SpmvPart p[kMaxPack];
    int32_t n;
};
typedef const __attribute__((address_space(4))) SpmvPart ConstSpmvPart;

template <int G>
__global__ void __launch_bounds__(kSpmvThreads, 8) spmv_parts_kernel(SpmvParts sp) {
    ConstSpmvPart *cp = (ConstSpmvPart *)&sp.p[0];
    int q = 0;
    for (int k = 1; k < sp.n; ++k)
        if (cp[k].wg_begin <= (int64_t)blockIdx.x) q = k;
    const int64_t i = cp[q].lo + ((blockIdx.x - cp[q].wg_begin) * kSpmvThreads + threadIdx.x) / G;
    const int g = threadIdx.x & (G - 1);
    const bool live = i < cp[q].hi;
    __shared__ double sh[kSpmvThreads / kWave][kWaveChunk];
    const int32_t *rp = cp[q].rp;
    const double s = row_sum<G, true>(cp[q].col, cp[q].val, cp[q].x, live ? rp[i] : 0, live ? rp[i + 1] : 0, g, sh);
    if (live && g == 0) cp[q].y[i] = s;
}

// ---------------------------------------------------------------------------
// Binned form.  What bounds the plain form is its gathers of x: each reads a
// 128-byte line through L1 (and, for an x beyond an XCD's 4 MB L2, mostly
// through the fabric) for 8 bytes of it.  Here every gather is an LDS access.
//
// The columns are cut into column blocks of kBinCols (an x segment of 128 KB
// in LDS), the rows into row blocks whose entries fit LDS, and the matrix's
// entries are copied once into column-block-major order, each column block's
// entries by row block (the bucket of row block r and column block c is a
// contiguous run).  A product is two launches:
//   multiply: each workgroup takes an equal share of that order, keeps the
//     current column block's x segment in LDS and streams
//     prod[i] = bval[i] * x[bcol[i]], all accesses contiguous;
//   sum: each workgroup takes a row block, copies its buckets' products to LDS
//     at the entries' places in the row order (dst) and adds each row's
//     products as the plain form does: lane g of G adds entries g, g + G, ...
//     in increasing k, then a fixed butterfly.
// The order inside a bucket is whatever the build left; the sums do not
// depend on it, nor on the row blocks, so y has the same bits for every
// partition count.  A row block with more entries than LDS holds keeps no
// buckets: the multiply launch sums its rows straight from the CSR arrays.
//
// An entry costs 8 + 2 bytes read and 8 written, then 8 + 2 read: 1.9 GB for
// 2^22 rows of 16.  Measured there: multiply 246 us (5.3 TB/s), sum 226 us
// (3.1 TB/s: see its comment), one-time copy 540 us; a form that walked one
// eighth of the columns per XCD took 841 us (its gathers 786, each a line from
// L2) and 5.3 ms for its copy, the plain form 1122 us.  2^20 rows of 16: 118
// us, plain 181; 2^19 rows: 72 us, plain 65, so the plain form stays the
// default below 2^20 columns.
// ---------------------------------------------------------------------------
constexpr int kBinShift = 14;
constexpr int kBinCols = 1 << kBinShift;  // x elements per column block (128 KB of LDS)
constexpr int kBinMaxRows = 1024;         // rows per row block
constexpr int kBinCap = 9600;             // products a row block may have in LDS (with its row pointers 80 KB: two per CU)
constexpr int kBinTarget = 7424;          // entries a row block is sized for at the matrix's mean row length
constexpr int kMulThreads = 1024;
constexpr int kMulGroups = 512;
constexpr int kSumRowThreads = 512;
constexpr int kSegments = 64;             // of row blocks, in the scan of the bucket sizes
constexpr int kPad = 64;                  // entries to which a column block's start is aligned
constexpr int kBig = 1024;                // entries beyond which a bucket is the whole workgroup's work
constexpr int kLongRow = 8192;            // entries beyond which a row is a workgroup's work

struct BinPart {
    const int32_t *rp;  // biased: rp[row]
    double *y;          // biased: y[row]
    int64_t r0, r1;
    int64_t blk;        // its first row block
};
struct BinParts {
    BinPart p[kMaxPack];
    int32_t n;
};
typedef const __attribute__((address_space(4))) BinPart ConstBinPart;

// Rows [lo, hi) of row block `blk`, and its partition's pointers.
struct BinBlock {
    const int32_t *rp;
    double *y;
    int64_t lo;
    int rows;
    int32_t e0, m;  // its first entry and entry count
};
__device__ __forceinline__ BinBlock bin_block(const BinParts &bp, int64_t blk, int rb) {
    ConstBinPart *cp = (ConstBinPart *)&bp.p[0];
    int q = 0;
    for (int k = 1; k < bp.n; ++k)
        if (cp[k].blk <= blk) q = k;
    BinBlock B;
    B.rp = cp[q].rp;
    B.y = cp[q].y;
    B.lo = cp[q].r0 + (blk - cp[q].blk) * rb;
    const int64_t left = cp[q].r1 - B.lo;
    B.rows = (int)(left < rb ? left : rb);
    B.e0 = B.rp[B.lo];
    B.m = B.rp[B.lo + B.rows] - B.e0;
    return B;
}

// group_sum for a lane count known at run time (the same in all lanes).
__device__ __forceinline__ double group_sum_of(double s, int G) {
    return G == 4 ? group_sum<4>(s) : G == 8 ? group_sum<8>(s) : group_sum<16>(s);
}

// Row block of a workgroup: the grid is a multiple of 8, and XCD x (workgroups
// b with b mod 8 = x) takes the x-th contiguous eighth of the blocks, so the
// lines that neighbouring blocks' buckets share are used in one L2.
__device__ __forceinline__ int64_t bin_order() {
    const int64_t b = blockIdx.x;
    return (b & 7) * (gridDim.x >> 3) + (b >> 3);
}

// ---- build ------------------------------------------------------------------
// cnt[blk][c] = entries of row block blk in column block c (none for a block
// beyond LDS)
__global__ void __launch_bounds__(512)
bin_count_kernel(BinParts bp, const int32_t *__restrict__ col, int rb, int nblk, int nc, uint16_t *__restrict__ cnt) {
    extern __shared__ int32_t hist[];
    const int64_t blk = bin_order();
    if (blk >= nblk) return;
    const BinBlock B = bin_block(bp, blk, rb);
    for (int c = threadIdx.x; c < nc; c += blockDim.x) hist[c] = 0;
    __syncthreads();
    if (B.m <= kBinCap)
        for (int32_t i = threadIdx.x; i < B.m; i += blockDim.x) atomicAdd(&hist[col[(int64_t)B.e0 + i] >> kBinShift], 1);
    __syncthreads();
    for (int c = threadIdx.x; c < nc; c += blockDim.x) cnt[blk * nc + c] = (uint16_t)hist[c];
}

// Totals of each column block over each of the kSegments segments of row
// blocks: segs[seg * nc + c].  Workgroups of 64 columns x 16 lanes.
__global__ void __launch_bounds__(1024)
bin_segments_kernel(const uint16_t *__restrict__ cnt, int nblk, int nc, int per, int32_t *__restrict__ segs) {
    __shared__ int32_t sh[16][64];
    const int c = blockIdx.x * 64 + (threadIdx.x & 63), j = threadIdx.x >> 6;
    const int lo = blockIdx.y * per, hi = lo + per < nblk ? lo + per : nblk;
    int32_t t = 0;
    if (c < nc)
        for (int b = lo + j; b < hi; b += 16) t += cnt[(int64_t)b * nc + c];
    sh[j][threadIdx.x & 63] = t;
    __syncthreads();
    if (j == 0 && c < nc) {
        for (int k = 1; k < 16; ++k) t += sh[k][threadIdx.x];
        segs[(int64_t)blockIdx.y * nc + c] = t;
    }
}

// One workgroup: the start of every column block, aligned to kPad entries
// (cbase[c]; cbase[nc] the end), and segs turned into the start of each
// segment within it; the counts of `over` are cleared.
__global__ void __launch_bounds__(1024)
bin_bases_kernel(int nc, int32_t *__restrict__ segs, int32_t *__restrict__ cbase, int32_t *__restrict__ over) {
    __shared__ int32_t sh[1024];
    int32_t before = 0;
    for (int c0 = 0; c0 < nc; c0 += 1024) {
        const int c = c0 + threadIdx.x;
        int32_t total = 0;
        if (c < nc)
#pragma unroll 16
            for (int g = 0; g < kSegments; ++g) total += segs[(int64_t)g * nc + c];
        const int32_t padded = (total + kPad - 1) / kPad * kPad;
        sh[threadIdx.x] = padded;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {
            const int32_t add = (int)threadIdx.x >= off ? sh[threadIdx.x - off] : 0;
            __syncthreads();
            sh[threadIdx.x] += add;
            __syncthreads();
        }
        int32_t at = before + sh[threadIdx.x] - padded;
        before += sh[1023];
        if (c < nc) {
            cbase[c] = at;
            for (int g0 = 0; g0 < kSegments; g0 += 16) {
                int32_t v[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) v[u] = segs[(int64_t)(g0 + u) * nc + c];
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    segs[(int64_t)(g0 + u) * nc + c] = at;
                    at += v[u];
                }
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        cbase[nc] = before;
        over[0] = over[1] = 0;
    }
}

// start[blk][c]: lane j of a column takes the j-th sixteenth of the segment.
__global__ void __launch_bounds__(1024)
bin_starts_kernel(const uint16_t *__restrict__ cnt, int nblk, int nc, int per, const int32_t *__restrict__ segs,
                  int32_t *__restrict__ start) {
    __shared__ int32_t sh[16][64];
    const int cl = threadIdx.x & 63, c = blockIdx.x * 64 + cl, j = threadIdx.x >> 6;
    const int lo = blockIdx.y * per, hi = lo + per < nblk ? lo + per : nblk;
    const int sub = (per + 15) / 16, b0 = lo + j * sub, b1 = b0 + sub < hi ? b0 + sub : hi;
    int32_t t = 0;
    if (c < nc)
        for (int b = b0; b < b1; ++b) t += cnt[(int64_t)b * nc + c];
    sh[j][cl] = t;
    __syncthreads();
    if (c >= nc) return;
    int32_t at = segs[(int64_t)blockIdx.y * nc + c];
    for (int k = 0; k < j; ++k) at += sh[k][cl];
    for (int b = b0; b < b1; ++b) {
        start[(int64_t)b * nc + c] = at;
        at += cnt[(int64_t)b * nc + c];
    }
}

// Copies a row block's entries into their buckets: value, column within the
// column block, place within the row block.  SORT: the entries are ordered by
// bucket in LDS first, so that a bucket is written by neighbouring lanes
// (2^22 rows of 16: 2.6 ms with each lane writing its own entry's bucket);
// the column blocks' counters then have to fit beside them.  A row block beyond
// LDS and its long rows go to the list `over` instead: over[0] and over[1] the
// counts, from over[2] on the blocks, from over[2 + nblk] on (block, row within
// it).
constexpr int kSortCols = 2048;
template <bool SORT>
__global__ void __launch_bounds__(1024)
bin_fill_kernel(BinParts bp, const int32_t *__restrict__ col, const double *__restrict__ val, int rb, int nblk, int nc,
                const int32_t *__restrict__ start, const uint16_t *__restrict__ cnt, double *__restrict__ bval,
                uint16_t *__restrict__ bcol, uint16_t *__restrict__ dst, int32_t *__restrict__ over) {
    extern __shared__ int32_t at[];  // next free entry of each bucket
    __shared__ double sval[SORT ? kBinCap : 1];
    __shared__ int32_t scol[SORT ? kBinCap : 1];
    __shared__ uint16_t sdst[SORT ? kBinCap : 1];
    __shared__ int32_t shift[SORT ? kSortCols : 1];  // a bucket's start in memory minus that in LDS
    __shared__ int32_t sums[1024 / kWave];
    const int64_t blk = bin_order();
    if (blk >= nblk) return;
    const BinBlock B = bin_block(bp, blk, rb);
    const int tid = threadIdx.x;
    if (B.m > kBinCap) {
        if (tid == 0) over[2 + atomicAdd(&over[0], 1)] = (int32_t)blk;
        for (int r = tid; r < B.rows; r += 1024)
            if (B.rp[B.lo + r + 1] - B.rp[B.lo + r] > kLongRow) {
                int32_t *at = over + 2 + nblk + 2 * atomicAdd(&over[1], 1);
                at[0] = (int32_t)blk;
                at[1] = r;
            }
        return;
    }
    if constexpr (!SORT) {
        for (int c = tid; c < nc; c += 1024) at[c] = start[blk * nc + c];
        __syncthreads();
        for (int32_t i = tid; i < B.m; i += 1024) {
            const int32_t c = col[(int64_t)B.e0 + i];
            const int32_t k = atomicAdd(&at[c >> kBinShift], 1);
            bval[k] = val[(int64_t)B.e0 + i];
            bcol[k] = (uint16_t)(c & (kBinCols - 1));
            dst[k] = (uint16_t)i;
        }
    } else {
        // exclusive scan of the bucket sizes, two columns per thread
        const int c = 2 * tid;
        const int32_t n0 = c < nc ? cnt[blk * nc + c] : 0, n1 = c + 1 < nc ? cnt[blk * nc + c + 1] : 0;
        int32_t t = n0 + n1;
#pragma unroll
        for (int m = 1; m < kWave; m <<= 1) {
            const int32_t o = __shfl_up(t, m, kWave);
            if ((tid & (kWave - 1)) >= m) t += o;
        }
        if ((tid & (kWave - 1)) == kWave - 1) sums[tid / kWave] = t;
        __syncthreads();
        for (int w = 0; w < tid / kWave; ++w) t += sums[w];
        const int32_t before = t - n0 - n1;
        if (c < nc) {
            at[c] = before;
            shift[c] = start[blk * nc + c] - before;
        }
        if (c + 1 < nc) {
            at[c + 1] = before + n0;
            shift[c + 1] = start[blk * nc + c + 1] - before - n0;
        }
        __syncthreads();
#pragma unroll 4
        for (int32_t i = tid; i < B.m; i += 1024) {
            const int32_t cc = col[(int64_t)B.e0 + i];
            const double x = val[(int64_t)B.e0 + i];
            const int32_t k = atomicAdd(&at[cc >> kBinShift], 1);
            sval[k] = x;
            scol[k] = cc;
            sdst[k] = (uint16_t)i;
        }
        __syncthreads();
        for (int32_t k = tid; k < B.m; k += 1024) {
            const int32_t cc = scol[k], to = k + shift[cc >> kBinShift];
            bval[to] = sval[k];
            bcol[to] = (uint16_t)(cc & (kBinCols - 1));
            dst[to] = sdst[k];
        }
    }
}

// ---- product ----------------------------------------------------------------
typedef uint16_t us4 __attribute__((ext_vector_type(4)));
typedef uint16_t us2u __attribute__((ext_vector_type(2), aligned(2)));

// The rows of row blocks beyond LDS, straight from the CSR arrays and in the same
// order, spread over all workgroups of the multiply launch: groups of G lanes a
// row, and for the rows of more than kLongRow entries a workgroup a row, which
// has the products of 16384 entries at a time in LDS and G lanes add them (2^20
// rows of 3 and one of 200,000: 16.0 ms when the row's block was one workgroup's
// work and its lanes took an entry at a time).
__device__ void bin_over_rows(const BinParts &bp, int rb, int nblk, int G, const int32_t *__restrict__ over,
                              const int32_t *__restrict__ col, const double *__restrict__ val,
                              const double *__restrict__ x, double *xs) {
    const int tid = threadIdx.x, per = kMulThreads / G, g = tid & (G - 1);
    const int slices = (rb + per - 1) / per;
    const int32_t *longs = over + 2 + nblk;
    for (int64_t u = blockIdx.x; u < (int64_t)over[0] * slices; u += gridDim.x) {
        const BinBlock B = bin_block(bp, over[2 + u / slices], rb);
        const int r = (int)(u % slices) * per + tid / G;
        int32_t kb = 0, ke = 0;
        if (r < B.rows) {
            kb = B.rp[B.lo + r];
            ke = B.rp[B.lo + r + 1];
        }
        const bool mine = r < B.rows && ke - kb <= kLongRow;
        const double s = group_sum_of(mine ? lane_sum<true>(col, val, x, kb, ke, g, G) : 0.0, G);
        if (mine && g == 0) B.y[B.lo + r] = s;
    }
    for (int32_t i = blockIdx.x; i < over[1]; i += gridDim.x) {
        const BinBlock B = bin_block(bp, longs[2 * i], rb);
        const int64_t row = B.lo + longs[2 * i + 1];
        const int64_t kb = B.rp[row], ke = B.rp[row + 1];
        double s = 0.0;
        for (int64_t base = kb; base < ke; base += kBinCols) {
            const int m = (int)(ke - base < kBinCols ? ke - base : kBinCols);
            __syncthreads();  // xs is free
#pragma unroll 8
            for (int k = tid; k < m; k += kMulThreads) xs[k] = val[base + k] * x[col[base + k]];
            __syncthreads();
            if (tid < G)
#pragma unroll 16
                for (int k = tid; k < m; k += G) s += xs[k];
        }
        if (tid < kWave) {
            s = group_sum_of(s, G);
            if (tid == 0) B.y[row] = s;
        }
    }
}

// prod = bval * x[bcol] over this workgroup's share of the column-block-major
// order.  The entries that align a column block's start hold anything: their
// column is masked to the segment, their product is never read.
__global__ void __launch_bounds__(kMulThreads)
bin_multiply_kernel(const int32_t *__restrict__ cbase, int nc, int64_t ncols, const double *__restrict__ x,
                    const double *__restrict__ bval, const uint16_t *__restrict__ bcol, double *__restrict__ prod,
                    BinParts bp, int rb, int nblk, int G, const int32_t *__restrict__ over,
                    const int32_t *__restrict__ col, const double *__restrict__ val) {
    __shared__ double xs[kBinCols];
    const int64_t total = cbase[nc];
    const int64_t per = ((total + gridDim.x - 1) / gridDim.x + kPad - 1) / kPad * kPad;
    int64_t i0 = blockIdx.x * per;
    const int64_t i1 = i0 + per < total ? i0 + per : total;
    int c = 0;
    for (int lo = 0, hi = nc - 1; lo <= hi;) {  // the last column block starting at or before i0
        const int mid = (lo + hi) >> 1;
        if (cbase[mid] <= i0) {
            c = mid;
            lo = mid + 1;
        } else {
            hi = mid - 1;
        }
    }
    for (; i0 < i1; ++c) {
        const int64_t end = cbase[c + 1] < i1 ? cbase[c + 1] : i1;
        if (end <= i0) continue;
        const double *seg = x + ((int64_t)c << kBinShift);
        const int64_t len = ncols - ((int64_t)c << kBinShift);
        __syncthreads();  // every wave is done with the previous segment
#pragma unroll 8
        for (int k = threadIdx.x; k < kBinCols; k += kMulThreads) xs[k] = k < len ? seg[k] : 0.0;
        __syncthreads();
        auto four = [&](int64_t i) {
            const us4 k = __builtin_nontemporal_load(reinterpret_cast<const us4 *>(bcol + i));
            const dvec2 a = __builtin_nontemporal_load(reinterpret_cast<const dvec2 *>(bval + i));
            const dvec2 b = __builtin_nontemporal_load(reinterpret_cast<const dvec2 *>(bval + i + 2));
            dvec2 p, q;
            p.x = a.x * xs[k.x & (kBinCols - 1)];
            p.y = a.y * xs[k.y & (kBinCols - 1)];
            q.x = b.x * xs[k.z & (kBinCols - 1)];
            q.y = b.y * xs[k.w & (kBinCols - 1)];
            *reinterpret_cast<dvec2 *>(prod + i) = p;
            *reinterpret_cast<dvec2 *>(prod + i + 2) = q;
        };
#pragma unroll 2
        for (int64_t i = i0 + threadIdx.x * 4; i < end; i += kMulThreads * 4) four(i);
        i0 = end;
    }
    if (over[0] != 0) bin_over_rows(bp, rb, nblk, G, over, col, val, x, xs);
}

// One row block per workgroup: LB lanes copy a bucket's products to LDS, two
// neighbours each, then G lanes add up a row.  What a bucket holds beyond its
// lanes' first two rounds is copied by a wave, or by the whole workgroup: the rows
// of a matrix with its columns near the diagonal have one or two buckets, over
// which 16 lanes took 2471 us a product (2^22 rows of 16 neighbours; 494 so, the
// plain form 274; 2^22 rows of 5: 762, 187 and 134).  The latency of its chain of
// loads (bucket table, then products, then the sums) bounds it, so all
// products of a block are in flight at once, and the row pointers with them.
// (Tried at 2^22 rows of 16, against 226 us: four workgroups of half the size
// per compute unit 230, smaller buckets 266, places read in row order during
// the sums 330, one bucket batch after the other 257, and a persistent walk
// that fetches the next block's table early, whose registers spilled, 395.)
template <int G, int LB>
__global__ void __launch_bounds__(kSumRowThreads)
bin_sum_kernel(BinParts bp, int rb, int nblk, int nc, const int32_t *__restrict__ start, const uint16_t *__restrict__ cnt,
               const double *__restrict__ prod, const uint16_t *__restrict__ dst) {
    __shared__ double v[kBinCap];
    __shared__ int32_t rps[kBinMaxRows + 1];
    constexpr int kSumWaves = kSumRowThreads / kWave;
    __shared__ __align__(16) int more[kSumWaves];  // a wave's buckets have entries left
    constexpr int kQ = kSumRowThreads / LB;  // buckets side by side
    constexpr int kU = 8;                    // and in each group's hands
    constexpr int kP = 2 * LB;               // entries a group takes at a time
    constexpr int kRp = (kBinMaxRows + kSumRowThreads) / kSumRowThreads;  // row pointers per thread
    const int64_t blk = bin_order();
    if (blk >= nblk) return;
    const int tid = threadIdx.x, sub = 2 * (tid & (LB - 1)), q = tid / LB;
    int most = 0;
    const int32_t *st = start + blk * nc;
    const uint16_t *ct = cnt + blk * nc;
    const BinBlock B = bin_block(bp, blk, rb);
    if (B.m > kBinCap) return;  // its rows are done (bin_over_rows)
    int32_t rp[kRp];
#pragma unroll
    for (int u = 0; u < kRp; ++u) {
        const int i = tid + u * kSumRowThreads;
        rp[u] = B.rp[B.lo + (i <= B.rows ? i : B.rows)];
    }
    for (int c0 = q; c0 < nc; c0 += kQ * kU) {
        int32_t at[kU], n[kU];
        dpair p[kU], p2[kU];
        us2u d[kU], d2[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            n[u] = at[u] = 0;
            if (c0 + u * kQ < nc) {
                n[u] = ct[c0 + u * kQ];
                at[u] = st[c0 + u * kQ];
            }
        }
        // the first 2 kP products of every bucket in flight at once (a pair
        // may reach one entry past its bucket: in the buffers, and not used)
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (sub < n[u]) {
                p[u] = *reinterpret_cast<const dpair *>(prod + at[u] + sub);
                d[u] = *reinterpret_cast<const us2u *>(dst + at[u] + sub);
            }
            if (sub + kP < n[u]) {
                p2[u] = *reinterpret_cast<const dpair *>(prod + at[u] + sub + kP);
                d2[u] = *reinterpret_cast<const us2u *>(dst + at[u] + sub + kP);
            }
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (sub < n[u]) v[d[u].x] = p[u].x;
            if (sub + 1 < n[u]) v[d[u].y] = p[u].y;
            if (sub + kP < n[u]) v[d2[u].x] = p2[u].x;
            if (sub + kP + 1 < n[u]) v[d2[u].y] = p2[u].y;
            most = n[u] > most ? n[u] : most;
        }
    }
#pragma unroll
    for (int u = 0; u < kRp; ++u)
        if (tid + u * kSumRowThreads <= B.rows) rps[tid + u * kSumRowThreads] = rp[u] - B.e0;
    const bool left = __any(most > 2 * kP);
    if ((tid & (kWave - 1)) == 0) more[tid / kWave] = left;
    __syncthreads();
    const int4 m0 = *reinterpret_cast<const int4 *>(&more[0]), m1 = *reinterpret_cast<const int4 *>(&more[4]);
    if (m0.x | m0.y | m0.z | m0.w | m1.x | m1.y | m1.z | m1.w) {  // entries past the first 2 kP of a bucket
        __shared__ uint16_t big[kBinCap / (2 * kP) + 1];
        __shared__ int nbig;
        if (tid == 0) nbig = 0;
        __syncthreads();
        for (int c = tid; c < nc; c += kSumRowThreads)
            if (ct[c] > 2 * kP) big[atomicAdd(&nbig, 1)] = (uint16_t)c;
        __syncthreads();
        auto copy = [&](int at, int m, int first, int step) {
#pragma unroll 4
            for (int i = 2 * kP + 2 * first; i < m; i += 2 * step) {
                const dpair p = *reinterpret_cast<const dpair *>(prod + at + i);
                const us2u d = *reinterpret_cast<const us2u *>(dst + at + i);
                v[d.x] = p.x;
                if (i + 1 < m) v[d.y] = p.y;
            }
        };
        for (int b = 0; b < nbig; ++b) {  // a wave takes a bucket's, all of them those of a large one
            const int c = big[b], m = ct[c];
            if (m > kBig)
                copy(st[c], m, tid, kSumRowThreads);
            else if (b % kSumWaves == tid / kWave)
                copy(st[c], m, tid & (kWave - 1), kWave);
        }
        __syncthreads();
    }
    const int g = tid & (G - 1);
    constexpr int kStep = kSumRowThreads / G, kR = 4;  // rows side by side, and in each group's hands
    for (int r0 = tid / G; r0 < B.rows; r0 += kStep * kR) {
        int32_t k[kR], ke[kR];
        double t[kR];
#pragma unroll
        for (int u = 0; u < kR; ++u) {
            const int r = r0 + u * kStep < B.rows ? r0 + u * kStep : r0;
            k[u] = rps[r] + g;
            ke[u] = rps[r + 1];
        }
#pragma unroll
        for (int u = 0; u < kR; ++u) t[u] = k[u] < ke[u] ? 0.0 + v[k[u]] : 0.0;
#pragma unroll
        for (int u = 0; u < kR; ++u) {
            for (int32_t i = k[u] + G; i < ke[u]; i += G) t[u] += v[i];
            t[u] = group_sum<G>(t[u]);
            if (g == 0 && r0 + u * kStep < B.rows) B.y[B.lo + r0 + u * kStep] = t[u];
        }
    }
}

BinParts bin_parts(const Launch *L, int n, int rb) {
    BinParts bp{};
    int64_t blk = 0;
    for (int k = 0; k < n; ++k) {
        const int64_t rows = L[k].hi[0] - L[k].lo[0];
        if (rows <= 0) continue;
        BinPart &d = bp.p[bp.n++];
        d.rp = (const int32_t *)L[k].a[0].ptr;
        d.y = (double *)L[k].a[4].ptr;
        d.r0 = L[k].lo[0];
        d.r1 = L[k].hi[0];
        d.blk = blk;
        blk += (rows + rb - 1) / rb;
    }
    return bp;
}

// Lanes per bucket: 16 take up to 64 entries at once, 64 up to 256.
int64_t bin_lanes(int64_t nc) { return kBinTarget > 48 * nc ? 64 : 16; }

unsigned bin_grid(int nblk) { return (unsigned)((nblk + 7) / 8 * 8); }

}  // namespace

// Lanes per row: about one entry each (2^19 rows: 4 entries a row 19 / 22 / 33
// us with 4 / 8 / 16 lanes, 8 entries 40 / 34 / 41, 16 entries 100 / 74 / 64).
int spmv_lanes(int64_t nnz, int64_t rows) {
    const int64_t mean = rows > 0 ? (nnz + rows - 1) / rows : 0;
    return mean > 8 ? 16 : mean > 4 ? 8 : 4;
}

// Rows per row block, by the mean row length.
static int64_t bin_rows(int64_t mean, int64_t nc) {
    // just past the change to 16 lanes a bucket, smaller blocks, whose buckets
    // seldom exceed the 64 entries that those take at once (2^22 rows of 16 over
    // 157 column blocks: 459 us, 466 without)
    const int64_t target = bin_lanes(nc) == 16 && 44 * nc < kBinTarget ? 44 * nc : kBinTarget;
    const int64_t rb = mean > 0 ? target / mean : kBinMaxRows;
    return rb < 16 ? 16 : rb > kBinMaxRows ? kBinMaxRows : rb;
}

// A binned product loads every column block's x and walks every bucket, whatever
// they hold.  It is faster from about 2^22 entries on (us, plain and binned; 2^20
// rows and columns, 2 / 4 / 8 entries a row: 30 and 42, 50 and 51, 93 and 75),
// where a column has an entry on average (2^22 columns, 2^16 / 2^18 rows of 16:
// 21 and 40, 74 and 57; 2^27 columns, 1000 rows of 16: 11 and 366) and a bucket
// four (2^24 columns, 2^22 rows of 4: 332 and 247; 2^26 columns, rows of 16, 1.8 a
// bucket: 1306 and 1301, and the copy takes 3 ms).
// A launch of some of the rows (a partition's, a box's) pays for all of x too, and
// asks for 5/8 of those entries, and three for four columns (a launch a partition,
// plain and binned: 2^21 rows of 6 over 4 187 and 146, over 8 198 and 224; 2^20 rows
// of 16 over 4 187 and 147, over 8 198 and 214, over 20 233 and 415; 2^22 rows of 16
// over 20 1186 and 810, over 64 1215 and 1740).
bool bin_pays(int64_t ncols, int64_t nnz, int64_t rows, int64_t launch_rows) {
    if (rows < 1) return false;
    const int64_t nc = (ncols + kBinCols - 1) >> kBinShift, rb = bin_rows((nnz + rows - 1) / rows, nc);
    const int64_t most = (int64_t)1 << 22, here = (int64_t)((double)nnz * ((double)launch_rows / (double)rows));
    return nnz >= most && nnz >= ncols && nnz >= 4 * nc * ((rows + rb - 1) / rb) &&
           (launch_rows >= rows || (8 * here > 5 * most && 4 * here >= 3 * ncols));
}

bool bin_geometry(int64_t ncols, int64_t nnz, int64_t rows, int64_t entries, const Launch *L, int n, BinBufs *bb) {
    *bb = BinBufs{};
    // the histogram of column blocks takes 4 bytes of LDS each (128 KB); row
    // blocks are sized by the mean row length of the whole matrix, and so are
    // the lanes of a row: neither depends on the partitions
    if (ncols < 1 || ncols > ((int64_t)kBinCols << 15) || n > kMaxPack) return false;
    const int64_t mean = (nnz + rows - 1) / (rows > 0 ? rows : 1);
    if (mean > kBinCap) return false;  // most row blocks would hold no buckets
    const int64_t nc = (ncols + kBinCols - 1) >> kBinShift, rb = bin_rows(mean, nc);
    bb->ncols = ncols;
    bb->nc = (int)nc;
    bb->rb = (int)rb;
    bb->lanes = spmv_lanes(nnz, rows);
    int64_t nblk = 0;
    for (int k = 0; k < n; ++k) {
        const int64_t r = L[k].hi[0] - L[k].lo[0];
        if (r > 0) nblk += (r + rb - 1) / rb;
    }
    if (nblk > (1 << 24) || entries + (int64_t)kPad * bb->nc > INT32_MAX) return false;
    bb->nblk = (int)nblk;
    const size_t cells = (size_t)nblk * bb->nc, cap = (size_t)entries + (size_t)kPad * bb->nc;
    const size_t bytes[kBinBuffers] = {cells * 4, cells * 2, (size_t)(bb->nc + 1) * 4, (size_t)kSegments * bb->nc * 4,
                                       cap * 8,   cap * 2,   cap * 2,                  cap * 8,
                                       (2 + (size_t)nblk + 2 * ((size_t)entries / kLongRow + 1)) * 4};
    for (int i = 0; i < kBinBuffers; ++i) bb->bytes[i] = bytes[i];
    return true;
}

hipError_t build_bins(const Launch *L, int n, const BinBufs &bb, hipStream_t s) {
    if (bb.nblk <= 0) return hipSuccess;
    const BinParts bp = bin_parts(L, n, bb.rb);
    const int32_t *col = (const int32_t *)L[0].a[1].ptr;
    const double *val = (const double *)L[0].a[2].ptr;
    const int per = (bb.nblk + kSegments - 1) / kSegments;
    const dim3 scan((unsigned)((bb.nc + 63) / 64), kSegments);
    const size_t lds = (size_t)bb.nc * 4;
    hipLaunchKernelGGL(bin_count_kernel, dim3(bin_grid(bb.nblk)), dim3(512), lds, s, bp, col, bb.rb, bb.nblk, bb.nc,
                       bb.cnt());
    hipLaunchKernelGGL(bin_segments_kernel, scan, dim3(1024), 0, s, bb.cnt(), bb.nblk, bb.nc, per, bb.segs());
    hipLaunchKernelGGL(bin_bases_kernel, dim3(1), dim3(1024), 0, s, bb.nc, bb.segs(), bb.cbase(), bb.over());
    hipLaunchKernelGGL(bin_starts_kernel, scan, dim3(1024), 0, s, bb.cnt(), bb.nblk, bb.nc, per, bb.segs(), bb.start());
    if (bb.nc <= kSortCols)
        hipLaunchKernelGGL((bin_fill_kernel<true>), dim3(bin_grid(bb.nblk)), dim3(1024), lds, s, bp, col, val, bb.rb,
                           bb.nblk, bb.nc, bb.start(), bb.cnt(), bb.bval(), bb.bcol(), bb.dst(), bb.over());
    else
        hipLaunchKernelGGL((bin_fill_kernel<false>), dim3(bin_grid(bb.nblk)), dim3(1024), lds, s, bp, col, val, bb.rb,
                           bb.nblk, bb.nc, bb.start(), bb.cnt(), bb.bval(), bb.bcol(), bb.dst(), bb.over());
    return hipGetLastError();
}

hipError_t launch_spmv_bins(const Launch *L, int n, const BinBufs &bb, hipStream_t s) {
    if (bb.nblk <= 0) return hipSuccess;
    const BinParts bp = bin_parts(L, n, bb.rb);
    const double *x = (const double *)L[0].a[3].ptr;
    hipLaunchKernelGGL(bin_multiply_kernel, dim3(kMulGroups), dim3(kMulThreads), 0, s, bb.cbase(), bb.nc, bb.ncols, x,
                       bb.bval(), bb.bcol(), bb.prod(), bp, bb.rb, bb.nblk, bb.lanes, bb.over(), (const int32_t *)L[0].a[1].ptr,
                       (const double *)L[0].a[2].ptr);
    const bool wide = bin_lanes(bb.nc) == 64;
#define BIN_SUM(G, LB)                                                                                                 \
    hipLaunchKernelGGL((bin_sum_kernel<G, LB>), dim3(bin_grid(bb.nblk)), dim3(kSumRowThreads), 0, s, bp, bb.rb, bb.nblk, \
                       bb.nc, bb.start(), bb.cnt(), bb.prod(), bb.dst())
#define BIN_SUM_LB(G)       \
    do {                    \
        if (wide)           \
            BIN_SUM(G, 64); \
        else                \
            BIN_SUM(G, 16); \
    } while (0)
    switch (bb.lanes) {
        case 4: BIN_SUM_LB(4); break;
        case 8: BIN_SUM_LB(8); break;
        default: BIN_SUM_LB(16); break;
    }
#undef BIN_SUM_LB
#undef BIN_SUM
    return hipGetLastError();
}

hipError_t launch_spmv_parts(const Launch *L, int n, hipStream_t s) {
    if (n > kMaxPack) return hipErrorInvalidValue;
    SpmvParts sp{};
    const int G = n > 0 ? L[0].cfg.tile : 16;
    int64_t wg = 0;
    for (int k = 0; k < n; ++k) {
        const int64_t rows = L[k].hi[0] - L[k].lo[0];
        if (rows <= 0) continue;
        sp.p[sp.n++] = {(const int32_t *)L[k].a[0].ptr, (const int32_t *)L[k].a[1].ptr, (const double *)L[k].a[2].ptr,
                        (const double *)L[k].a[3].ptr,  (double *)L[k].a[4].ptr,        L[k].lo[0],
                        L[k].hi[0],                     wg};
        wg += (rows * G + kSpmvThreads - 1) / kSpmvThreads;
    }
    if (wg == 0) return hipSuccess;
    if (wg > INT32_MAX) return hipErrorInvalidValue;
    switch (G) {
        case 4: hipLaunchKernelGGL(spmv_parts_kernel<4>, dim3((unsigned)wg), dim3(kSpmvThreads), 0, s, sp); break;
        case 8: hipLaunchKernelGGL(spmv_parts_kernel<8>, dim3((unsigned)wg), dim3(kSpmvThreads), 0, s, sp); break;
        default: hipLaunchKernelGGL(spmv_parts_kernel<16>, dim3((unsigned)wg), dim3(kSpmvThreads), 0, s, sp); break;
    }
    return hipGetLastError();
}

hipError_t launch_spmv(const Launch &L, hipStream_t s) {
    const int64_t n = L.hi[0] - L.lo[0];
    if (n <= 0) return hipSuccess;
    // configuration: tile = lanes per row (4, 8 or 16), order 2 = non-temporal
    // col/val loads
    const int G = L.cfg.tile;
    const bool nt = L.cfg.order == 2;
    const int64_t rows_per_block = kSpmvThreads / G;
    const unsigned nb = (unsigned)((n + rows_per_block - 1) / rows_per_block);
#define SPMV_ARGS                                                                                                  \
    (const int32_t *)L.a[0].ptr, (const int32_t *)L.a[1].ptr, (const double *)L.a[2].ptr, (const double *)L.a[3].ptr, \
        (double *)L.a[4].ptr, L.lo[0], L.hi[0]
#define SPMV_LAUNCH(GG)                                                                                 \
    do {                                                                                                \
        if (nt)                                                                                         \
            hipLaunchKernelGGL((spmv_kernel<GG, true>), dim3(nb), dim3(kSpmvThreads), 0, s, SPMV_ARGS); \
        else                                                                                            \
            hipLaunchKernelGGL((spmv_kernel<GG, false>), dim3(nb), dim3(kSpmvThreads), 0, s, SPMV_ARGS); \
    } while (0)
    switch (G) {
        case 4: SPMV_LAUNCH(4); break;
        case 16: SPMV_LAUNCH(16); break;
        default: SPMV_LAUNCH(8); break;
    }
#undef SPMV_LAUNCH
#undef SPMV_ARGS
    return hipGetLastError();
}

}  // namespace jk
