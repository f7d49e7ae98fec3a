// Internal interface between the runtime (runtime.cpp) and the HIP loop
// bodies (k_*.hip).  Not part of the public ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace jk {

// Workgroups of `threads` threads that one launch takes: its threads along a
// dimension stay below 2^32.
constexpr int64_t max_groups(int threads) { return (((int64_t)1 << 32) - 1) / threads; }

// One argument as a kernel sees it: `ptr` is the device address of global
// row 0 of the array *as if* the slab started there (slab pointer minus
// slab_lo rows), so kernels index with global row numbers; only rows
// [slab_lo, slab_hi) may be touched.  For a 2-D array partitioned along
// dim 1 the slab holds columns [slab_lo, slab_hi) of every row, `ptr` is
// the slab pointer minus slab_lo elements, and element (i, j) sits at
// ptr + i*row_elems + j.
struct Arg {
    const void *ptr;       // biased pointer (see above)
    int64_t slab_lo, slab_hi;
    int64_t row_elems;     // elements per row of dim 0 (the slab's width when split along dim 1)
};

struct Cfg {
    int bx, by, tile, vec, persistent, order, march, rows;
    int odd;  // set with vec = 2 by the defaults: pairs in rows of odd length (a caller's own vec = 2 there is refused)
};

// Write-through targets of a stencil launch: rows [lo, hi) of dim 0 that the
// launch writes are also stored at `ptr` (biased like Arg::ptr), which is
// another partition's slab holding those rows as halo.
struct Mirror {
    double *ptr;
    int64_t lo, hi;
};
struct Mirrors {
    Mirror m[2];
    int n;
};
// Column mirrors (a 2-D array split along dim 1): [lo, hi) are the columns
// the holder slab keeps, pitch its row length in elements, and ptr is biased
// so that ptr[row * pitch + column] is global (row, column).
struct ColMirror {
    double *ptr;
    int64_t lo, hi, pitch;
};
struct ColMirrors {
    ColMirror m[2];
    int n;
};

// One partition's launch of one loop nest.
struct Launch {
    int kind;
    int ndim;
    int64_t lo[3], hi[3];       // iteration box (dim 0 already clipped to the partition)
    int64_t ext[4];             // extents of the first argument's array
    Arg a[6];
    int nargs;
    double scalars[4];
    Cfg cfg;
    int part_dim;     // the dimension the arrays are split along (0, or 1 for 2-D column slabs)
    Mirrors mir;      // stencil kinds only
    ColMirrors cmir;  // JACOBI2D on arrays split along dim 1 (mir is then empty)
    int64_t own_lo, own_hi;    // owner rows of a FILTERED output (writes elsewhere are dropped)
    int64_t own2_lo, own2_hi;  // owner rows of a second FILTERED output (PRED_CHAIN's b)
    // reductions: workgroup partials go to `wg_partials` (capacity
    // `wg_capacity` doubles); the finaliser writes their ordered sum to
    // `part_out`.  Both null when the loop reduces nothing.
    double *wg_partials;
    int64_t wg_capacity;
    double *part_out;
    // set when the loop's partitions are all in this launch (or pack): the sum
    // over them, written by the finaliser; `total_host`, pinned, may be null
    double *total, *total_host;
    unsigned *ticket;  // for packed launches: zero, and zero again when the finaliser ends
    bool streamed;      // other loops' arrays pass through the caches between its runs
    int64_t part_rows;  // iterations along dim 0 of the largest partition (for defaults)
    int beside;         // launches of the same loop on streams of their own, this one among them
};

// Launches the loop body (and, for reductions, the per-partition
// finaliser) on `s`.  Returns hipErrorInvalidValue for a configuration the
// body does not support; the runtime validates shapes before calling.
hipError_t launch_loop(const Launch &L, hipStream_t s);

// Checks a configuration for a loop without launching; returns 0 if legal.
int check_config(const Launch &L);

// Bytes of a stencil's two arrays up to which they are taken to live in the
// 256 MB memory-side cache from one sweep to the next: their outputs are then
// stored normally instead of non-temporally, and their tiles walked XCD-aware.
// Measured (us a sweep, non-temporal row-major / normal XCD-aware): Jacobi
// 2048^2 16.2 / 11.9, 4099x3001 40.1 / 30.1, 4150x4100 (272 MB) 51.4 / 45.6,
// 4200^2 (282 MB) 51.9 / 54.5, 5000^2 69.0 / 73.7; heat 128^3 10.0 / 9.1, 256^3
// (268 MB) 51 / 43, 301x303x305 (445 MB) 105 / 114.
constexpr int64_t kCacheBytes = 264 << 20;
constexpr int64_t kWgCapacity = 1 << 16;  // workgroup partials a stream's reduction holds
inline int64_t array_bytes(const Launch &L) {
    int64_t n = 8;
    for (int i = 0; i < 4; ++i)
        if (L.ext[i] > 0) n *= L.ext[i];
    return n;
}
inline bool cache_resident(const Launch &L) { return !L.streamed && 2 * array_bytes(L) <= kCacheBytes; }

// Fills in defaults for zero fields of a configuration.
Cfg default_config(int kind, const Launch &L, Cfg c);

// Reduction combine: out[0] = sum of partials[idx[k]] for k = 0..n-1 in
// that order (idx lists the reducing partitions in partition order; each
// partition's finaliser writes partials[p]).
struct CombineList {
    int n;
    int idx[64];
};
hipError_t launch_combine(const double *partials, const CombineList &list, double *out, double *host, hipStream_t s);

// One loop of a persistent task group: a stencil sweep cut into tiles of
// 256 threads, bx along a row and 256/bx row groups (2-D: of `tile` rows each;
// 3-D: of one row each through `tile` planes).
struct PTask {
    int32_t kind;  // JACC_LOOP_JACOBI2D or JACC_LOOP_HEAT3D
    int32_t vec, tile, march, bx;
    int32_t order;  // merged loops only
    const double *in;
    double *out;
    int64_t e1, e2;  // extents of dims 1 and 2 (2-D: e1 = row length)
    int64_t lo[3], hi[3];
    int64_t col0;
    double alpha;
    int64_t gx, gy, gz;
    int64_t ntiles, tile_begin;
    Mirrors mir;
};
constexpr int kPersistentThreads = 256;

// Builds the task record of a launch (false if the kind cannot run inside
// the persistent kernel).
bool make_task(const Launch &L, PTask *t);

// Workgroups of a persistent launch over `tiles` tiles (one per tile).
int64_t persistent_grid(int64_t tiles, bool jacobi_only);

// Launches the persistent kernel with `grid` workgroups over `ntasks` device
// task records whose tiles total `tiles` (jacobi_only: every task is a
// Jacobi sweep, which selects the variant without the heat bodies; nt: with
// non-temporal stores, for tasks that together exceed kCacheBytes).
hipError_t launch_persistent(const PTask *tasks, int ntasks, int64_t tiles, int64_t grid, bool jacobi_only, bool nt,
                             hipStream_t s);

// Independent stencil loops of a batch in one launch ("merged"): each has its own
// default shape (256 threads, cfg.bx along a row) and its tiles a run of
// workgroups starting at a multiple of 8.  make_merged gives a loop's task, with
// tile_begin unset; false: a loop this cannot run (mirrors, a filtered output, a
// shape of the caller's).  `workgroups` is the total with every run rounded up.
bool make_merged(const Launch &L, PTask *t);
hipError_t launch_merged(const PTask *tasks, int ntasks, int64_t workgroups, bool nt, hipStream_t s);

// The partitions of one eager stencil (or SUM) loop in one launch ("packed"): the
// launches of its partitions (the same kind, configuration and box apart
// from the dim-0 range, pointers, mirrors and reduction target), at most
// kMaxPack.  Each partition's tiles take a run of workgroups starting at a
// multiple of 8, so the XCD-aware tile orders hold within it.  With a
// residual, partition p's workgroup partials go to wg_partials + (its first
// tile among all partitions') and one more launch writes every partition's
// ordered sum to its part_out and their total to the first one's total.  Returns hipErrorInvalidValue
// for more than kMaxPack launches or more than wg_capacity partials.
constexpr int kMaxPack = 16;
hipError_t launch_parts(const Launch *L, int n, double *wg_partials, int64_t wg_capacity, hipStream_t s);

// `steps` (odd, at most kChainMax) Jacobi sweeps of the box [lo, hi) from the
// `in` array to the `out` array of the partitions' slabs, which split the rows
// [0, ny) in order; afterwards `out` holds the last sweep's result, in the rows
// [lo, hi) of each partition and in its mirrors, as after that sweep alone.
constexpr int kChainMax = 9;
struct ChainPart {
    const double *in;  // biased so that in[row * nx + column] is global (row, column)
    double *out;
    int64_t lo, hi;  // the rows the partition owns
    Mirrors mir;     // of `out`
};
struct Chain {
    ChainPart p[kMaxPack];
    int32_t n;
    int64_t ny, nx, lo[2], hi[2];
};
hipError_t launch_steps(const Chain &ch, int steps, hipStream_t s);
// Whether steps over that box gain by sharing launches.
bool steps_share(const Chain &ch);

// Workgroup partials a packed heat launch with a residual writes.
int64_t parts_partials(const Launch *L, int n);

// Segments base[off[k] .. off[k] + n[k]) of workgroup partials, k < count.
struct Segments {
    int64_t off[kMaxPack], n[kMaxPack];
    double *out[kMaxPack];
    int32_t count;
};
// Finaliser and combine in one launch: *total (and *host, unless null) = the
// segments' sums, each in the finaliser's order, added in segment order.  Each segment's sum also goes
// to its `out`, and `ticket` is used, when there are several.
hipError_t launch_total(const double *base, const Segments &seg, unsigned *ticket, double *total, double *host,
                        hipStream_t s);
// The partitions of one SUM loop in one launch, then their finalisers (the
// same bits as a launch per partition).
hipError_t launch_sum_parts(const Launch *L, int n, double *wg_partials, int64_t wg_capacity, hipStream_t s);

// Number of workgroups the loop's reduction writes partials for (for
// sizing; <= wg_capacity is required).
int64_t reduction_workgroups(const Launch &L);

// ---- per-kind launchers (k_*.hip) -----------------------------------------
hipError_t launch_jacobi2d(const Launch &L, hipStream_t s);
hipError_t launch_heat3d(const Launch &L, hipStream_t s);
int64_t heat3d_workgroups(const Launch &L);
hipError_t launch_sum(const Launch &L, hipStream_t s);
int64_t sum_workgroups(const Launch &L);
hipError_t launch_finalise(const double *partials, int64_t n, double *out, hipStream_t s);
// The sum of one launch's n workgroup partials: to L.total when that is set,
// else to L.part_out.
hipError_t launch_result(const Launch &L, int64_t n, hipStream_t s);
hipError_t launch_gemm(const Launch &L, hipStream_t s);
hipError_t launch_spmv(const Launch &L, hipStream_t s);
// The plain products of at most kMaxPack partitions in one launch, each on its
// own slabs (cfg.tile of the first: lanes per row).
hipError_t launch_spmv_parts(const Launch *L, int n, hipStream_t s);

// Binned SpMV: the device copy of the matrix rows of one or more partitions'
// launches, its geometry and buffers (k_spmv.hip).
constexpr int kBinBuffers = 9;
struct BinBufs {
    int64_t ncols;
    int nc, rb, nblk, lanes;  // column blocks, rows per row block, row blocks, lanes per row
    size_t bytes[kBinBuffers];
    void *mem[kBinBuffers];
    int32_t *start() const { return (int32_t *)mem[0]; }   // [row block][column block]: a bucket's first entry
    uint16_t *cnt() const { return (uint16_t *)mem[1]; }   // [row block][column block]: its entries
    int32_t *cbase() const { return (int32_t *)mem[2]; }   // a column block's first entry
    int32_t *segs() const { return (int32_t *)mem[3]; }    // scratch of the build's scan
    double *bval() const { return (double *)mem[4]; }      // the entries: value,
    uint16_t *bcol() const { return (uint16_t *)mem[5]; }  // column within its block,
    uint16_t *dst() const { return (uint16_t *)mem[6]; }   // place in its row block
    double *prod() const { return (double *)mem[7]; }      // products of the last multiply
    int32_t *over() const { return (int32_t *)mem[8]; }    // the row blocks beyond LDS and their long rows
};
// Lanes per row by the mean row length of the whole matrix (not by
// partition: the lanes decide the order of a row's sum).
int spmv_lanes(int64_t nnz, int64_t rows);
// Whether the binned form is the faster one for a launch of `launch_rows` of a
// matrix's rows (by default, from 2^20 columns on).
bool bin_pays(int64_t ncols, int64_t nnz, int64_t rows, int64_t launch_rows);
// Geometry for a matrix of `rows` rows and `nnz` entries, and the buffer sizes of
// a copy of the launches' rows, which hold `entries` of them (false: this form
// does not take the matrix).
bool bin_geometry(int64_t ncols, int64_t nnz, int64_t rows, int64_t entries, const Launch *L, int n, BinBufs *bb);
// Both read col, val and x through the first launch's arguments (every
// partition's replica holds the same values).
hipError_t build_bins(const Launch *L, int n, const BinBufs &bb, hipStream_t s);
hipError_t launch_spmv_bins(const Launch *L, int n, const BinBufs &bb, hipStream_t s);
hipError_t launch_scatter(const Launch &L, hipStream_t s);
hipError_t launch_chain(const Launch &L, hipStream_t s);

// Fills `height` lines of `width_bytes` bytes, `pitch_bytes` apart from
// `base`, with 0xFF bytes (k_fill.hip; all three multiples of 4).
hipError_t launch_poison(void *base, size_t pitch_bytes, size_t width_bytes, int64_t height, hipStream_t s);

// ---- learned cost model (k_mlp.hip) ----------------------------------------
constexpr int kMlpHidden = 64;
constexpr int kMlpMaxFeatures = 16;

// Gradient partials of a training step: one set per workgroup, which walks
// every kMlpGroups-th tile of 16 samples (64 sets of 37 KB: minibatches up
// to 1024 samples spread one tile to a workgroup, and their sum stays a
// short loop over independent loads).
constexpr int kMlpGroups = 64;

// Device buffers of one model: parameters, Adam moments, gradient, feature
// scaler, the workgroups' gradient partials and squared-error sums, and the
// predictions of `cap` samples.
struct MlpBufs {
    int F = 0, cap = 0;
    float *params = nullptr, *m = nullptr, *v = nullptr, *grad = nullptr, *mu = nullptr, *sd = nullptr;
    float *yhat = nullptr;
    float *part = nullptr;    // kMlpGroups x parameters
    double *sqerr = nullptr;  // kMlpGroups
    float *loss = nullptr;    // loss of each training step
};
int mlp_nparams(int F);
// Forward pass of n samples.
hipError_t mlp_forward(const MlpBufs &B, const float *X, int n, float *yhat, hipStream_t s);
// Forward and backward pass of n samples (rows idx[b] of X and y, or row b
// when idx is null): the parameter gradient (B.grad) and the mean squared
// error (*loss), and for t > 0 the Adam step t (1-based) on it.
hipError_t mlp_train(const MlpBufs &B, const float *X, const float *y, const int *idx, int n, int t, float lr,
                     float *loss, hipStream_t s);
// One Adam step (t is 1-based) on the last gradient.
hipError_t mlp_adam(const MlpBufs &B, int t, float lr, hipStream_t s);

}  // namespace jk
