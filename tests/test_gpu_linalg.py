"""GPU parity of the reduction, contraction and SpMV loop bodies against the
CPU oracle, at the stated tolerances (sum: 1e-13 relative to the sum of
magnitudes; GEMM: 1e-12 * ||A||_F ||B||_F in Frobenius norm, exact for
integer-valued inputs; SpMV: 1e-13 relative to each row's sum of
magnitudes)."""
import math

import numpy as np
import pytest

import oracle
from paper_2110_14340_amd import inputs, jacc
from gpu_util import context, say

pytestmark = pytest.mark.gpu


# ------------------------------------------------------------------ sum
@pytest.mark.parametrize("n,K", [(1, 1), (1000, 1), (1000, 3), (123_457, 4), (2_000_003, 8), (2_000_003, 16),
                                 (123_457, 20)])
def test_sum_small(n, K):
    say(f"sum n={n} K={K}")
    x = inputs.uniform(n, seed=n, lo=-1.0, hi=1.0)
    ref = oracle.sum_(x)
    mag = float(np.abs(x).sum())
    with context(K) as c:
        c.enter(x)
        s = c.sum(x)
        sq = c.sum(x, squares=True)
    assert abs(s - ref) <= 1e-13 * mag
    assert abs(sq - oracle.sum_(x, squares=True)) <= 1e-13 * float((x * x).sum())


def test_sum_512_cubed_k1_k4():
    say("sum 512^3 K=1,4")
    x = inputs.uniform((512, 512, 512), seed=7)
    ref = oracle.sum_(x)
    for K in (1, 4):
        with context(K) as c:
            c.enter(x)
            s = c.sum(x)
        assert abs(s - ref) <= 1e-13 * ref


@pytest.mark.parametrize("n,K", [(2_000_003, 3), (1 << 24, 8), (5_000_000, 16)])
def test_sum_packed_partitions_equal_a_launch_per_partition(n, K):
    """One launch over all partitions (the default) and a launch per
    partition on its own stream add in the same order: the sums are
    bit-identical, and within the oracle's bound."""
    say(f"sum packed vs per-partition n={n} K={K}")
    x = inputs.uniform(n, seed=n + K, lo=-1.0, hi=1.0)
    got = []
    for flags in (0, jacc.INIT_NO_PACK):
        with context(K, flags) as c:
            c.enter(x)
            got.append((c.sum(x), c.sum(x, squares=True)))
    assert got[0] == got[1]
    assert abs(got[0][0] - oracle.sum_(x)) <= 1e-13 * float(np.abs(x).sum())


def test_sum_integer_exact_and_deferred_slots():
    say("sum integer exact")
    x = (np.arange(1 << 20) % 1024).astype(np.float64)
    with context(2) as c:
        c.enter(x)
        c.sum(x, slot=5, sync=False)
        c.sum(x, squares=True, slot=6, sync=False)
        vals = c.reductions(5, 2)
    assert vals[0] == (1 << 10) * (1023 * 1024 // 2)
    assert vals[1] == (1 << 10) * sum(i * i for i in range(1024))


# ------------------------------------------------------------------ GEMM
def _gemm_dev(A, B, K, slab=0, threads=0, whole=True):
    C = np.zeros((A.shape[0], B.shape[1]))
    with context(K) as c:
        c.enter(A)
        c.enter(B, whole=whole)
        c.enter(C, clause=jacc.CREATE)
        c.gemm(A, B, C, cfg=jacc.config(tile=slab, bx=threads) if (slab or threads) else None)
        c.exit(C, jacc.COPYOUT)
    return C


@pytest.mark.parametrize("M,N,L,K", [(64, 64, 16, 1), (200, 150, 130, 1), (200, 150, 130, 3),
                                     (129, 257, 33, 2), (1, 5, 7, 1), (300, 17, 1000, 4)])
def test_gemm_small_frobenius_and_integer_exact(M, N, L, K):
    say(f"gemm {M}x{N}x{L} K={K}")
    A, B = inputs.gemm_inputs(M, N, L, seed=3)
    ref = oracle.gemm(A, B)
    Ai, Bi = inputs.gemm_inputs(M, N, L, seed=4, integer=True)
    for slab, threads in ((16, 256), (32, 256), (16, 512), (32, 512)):
        C = _gemm_dev(A, B, K, slab, threads)
        assert np.linalg.norm(C - ref) <= 1e-12 * np.linalg.norm(A) * np.linalg.norm(B)
        assert np.array_equal(_gemm_dev(Ai, Bi, K, slab, threads), oracle.gemm(Ai, Bi))


def test_gemm_4096_full_frobenius_and_integer_exact():
    """C = A*B at 4096^3 against the oracle over every element of C:
    Frobenius-norm bound for uniform inputs, exact equality for
    integer-valued inputs (whose products and sums are all exact)."""
    n = 4096
    A, B = inputs.gemm_inputs(n, n, n, seed=3)
    say(f"oracle: gemm 4096^3 on {oracle.threads()} host threads")
    ref = oracle.gemm_mt(A, B)
    bound = 1e-12 * np.linalg.norm(A) * np.linalg.norm(B)
    C1 = _gemm_dev(A, B, 1)
    say(f"  K=1 Frobenius error {np.linalg.norm(C1 - ref):.3e} (bound {bound:.3e})")
    assert np.linalg.norm(C1 - ref) <= bound
    C4 = _gemm_dev(A, B, 4)
    assert np.array_equal(C1, C4)  # no split-k: partitioning never changes an element's sum order
    assert np.linalg.norm(C4 - ref) <= bound
    assert np.array_equal(C1, _gemm_dev(A, B, 1, 32))  # nor does the k-slab depth
    assert np.array_equal(C1, _gemm_dev(A, B, 1, 16, 256))  # nor the workgroup size
    del C1, C4, ref
    Ai, Bi = inputs.gemm_inputs(n, n, n, seed=5, integer=True)
    say("  integer-valued inputs")
    ref_i = oracle.gemm_mt(Ai, Bi)
    assert np.array_equal(_gemm_dev(Ai, Bi, 4), ref_i)


# ------------------------------------------------------------------ SpMV
def _spmv_dev(rp, col, val, x, K, cfg=None, whole=True):
    y = np.zeros(rp.size - 1)
    with context(K) as c:
        c.enter(rp, halo=(1, 1))
        c.enter(col, whole=whole)
        c.enter(val, whole=whole)
        c.enter(x, whole=whole)
        c.enter(y, clause=jacc.CREATE)
        c.spmv(rp, col, val, x, y, cfg=cfg)
        c.exit(y, jacc.COPYOUT)
    return y


def _row_bound(rp, col, val, x):
    absx = np.abs(val * x[col])
    cs = np.concatenate([[0.0], np.cumsum(absx)])
    return cs[rp[1:]] - cs[rp[:-1]]


@pytest.mark.parametrize("n,K", [(1, 1), (100, 1), (1000, 3), (5000, 4), (5000, 16), (5000, 20)])
def test_spmv_small(n, K):
    say(f"spmv n={n} K={K}")
    rp, col, val, x = inputs.csr_matrix(n, n, 16, seed=8)
    ref = oracle.spmv_csr(rp, col, val, x)
    y = _spmv_dev(rp, col, val, x, K)
    assert np.all(np.abs(y - ref) <= 1e-13 * _row_bound(rp, col, val, x))
    rpi, coli, vali, _ = inputs.csr_matrix(n, n, 16, seed=9, integer_values=True)
    xi = inputs.int_valued(n, seed=10, lo=-10, hi=10)
    ref_i = oracle.spmv_csr(rpi, coli, vali, xi)
    assert np.array_equal(_spmv_dev(rpi, coli, vali, xi, K), ref_i)
    # lanes per row; order 2: non-temporal col/val loads; order 4: column bands (by per XCD)
    for lanes, order, by, rows in ((4, 1, 0, 0), (16, 1, 0, 0), (8, 2, 0, 0), (4, 2, 0, 0), (16, 4, 1, 0), (8, 4, 2, 0),
                                   (4, 4, 8, 0), (1, 4, 1, 0), (2, 4, 2, 0), (1, 4, 1, 2), (1, 4, 2, 4)):
        cfg = jacc.config(tile=lanes, order=order, by=by, rows=rows)
        assert np.all(np.abs(_spmv_dev(rp, col, val, x, K, cfg) - ref) <= 1e-13 * _row_bound(rp, col, val, x))
        assert np.array_equal(_spmv_dev(rpi, coli, vali, xi, K, cfg), ref_i)


@pytest.mark.parametrize("n,K,draws", [(3000, 1, 40), (20000, 3, 70)])
def test_spmv_rows_longer_than_the_lane_group(n, K, draws):
    """Rows of up to `draws` entries: every lane of a row group adds several
    terms in increasing k."""
    say(f"spmv n={n} K={K} up to {draws} entries per row")
    rp, col, val, x = inputs.csr_matrix(n, n, draws, seed=11)
    ref = oracle.spmv_csr(rp, col, val, x)
    bound = 1e-13 * _row_bound(rp, col, val, x)
    for lanes, order, by, rows in ((4, 2, 0, 0), (8, 1, 0, 0), (16, 2, 0, 0), (16, 4, 1, 0), (8, 4, 4, 0), (1, 4, 1, 0),
                                   (2, 4, 2, 0), (1, 4, 1, 4), (1, 4, 2, 2)):
        y = _spmv_dev(rp, col, val, x, K, jacc.config(tile=lanes, order=order, by=by, rows=rows))
        assert np.all(np.abs(y - ref) <= bound)


def test_banded_spmv_rebuilds_after_the_matrix_changes():
    """The banded copy is built at the first product and reused; new values
    (update to the device) and a new row_ptr/col (re-entered arrays) give
    products of the new matrix."""
    say("banded spmv reuse and rebuild")
    n = 30000
    rp, col, val, x = inputs.csr_matrix(n, n, 16, seed=12)
    cfg = jacc.config(tile=16, order=4, by=2)
    y = np.zeros(n)
    with context(3) as c:
        for arr in (col, val, x):
            c.enter(arr, whole=True)
        c.enter(rp, halo=(1, 1))
        c.enter(y, clause=jacc.CREATE)
        for step in range(3):
            if step == 2:
                val[:] = -2.0 * val
                c.update(val, jacc.UPDATE_DEVICE)
            c.spmv(rp, col, val, x, y, cfg=cfg)
            c.update(y, jacc.UPDATE_HOST)
            ref = oracle.spmv_csr(rp, col, val, x)
            assert np.all(np.abs(y - ref) <= 1e-13 * _row_bound(rp, col, val, x)), step
        c.exit(y)


def test_spmv_2_22_rows_k1_k4_every_row():
    say("spmv 2^22 rows K=1,4, every row against the oracle")
    n = 1 << 22
    rp, col, val, x = inputs.csr_matrix(n, n, 16, seed=4)
    ref = oracle.spmv_csr_mt(rp, col, val, x)
    bound = 1e-13 * _row_bound(rp, col, val, x)
    y1 = _spmv_dev(rp, col, val, x, 1)
    y4 = _spmv_dev(rp, col, val, x, 4)
    assert np.array_equal(y1, y4)  # each row's sum order is fixed by the lanes-per-row layout
    bad = np.flatnonzero(np.abs(y4 - ref) > bound)
    assert bad.size == 0, f"{bad.size} rows outside the bound, first {bad[:5]}"
    for by in (1, 2):
        say(f"  column-banded form, {8 * by} bands, K=1 and 4")
        cfg = jacc.config(tile=16, order=4, by=by)
        b1 = _spmv_dev(rp, col, val, x, 1, cfg)
        assert np.array_equal(_spmv_dev(rp, col, val, x, 4, cfg), b1)  # band boundaries do not depend on K
        bad = np.flatnonzero(np.abs(b1 - ref) > bound)
        assert bad.size == 0, f"{bad.size} banded rows outside the bound, first {bad[:5]}"
    say("  col, val and x as one shared read-only copy, K=4 (default and banded forms)")
    assert np.array_equal(_spmv_dev(rp, col, val, x, 4, whole=jacc.SHARED), y4)
    assert np.array_equal(_spmv_dev(rp, col, val, x, 4, cfg, whole=jacc.SHARED), b1)  # b1: the last banded form


# ------------------------------------------------------------------ predicate-filtered scatter
@pytest.mark.parametrize("n,K", [(1000, 1), (1000, 3), (100_003, 4), (1 << 22, 8)])
def test_filtered_scatter_matches_oracle(n, K):
    say(f"scatter n={n} K={K}")
    x = inputs.uniform(n, seed=n % 97, lo=-2, hi=2)
    idx = np.random.default_rng(n % 89).permutation(n).astype(np.int32)
    out = inputs.uniform(n, seed=5)
    ref = oracle.scatter_sq(x, idx, out)
    o = out.copy()
    with context(K) as c:
        c.enter(x, whole=True)
        c.enter(idx, whole=True)
        c.enter(o)
        c.scatter_sq(x, idx, o)
        c.exit(o)
    assert np.array_equal(o, ref)


@pytest.mark.parametrize("M,N,L,K", [(200, 150, 130, 3), (300, 17, 1000, 4)])
def test_gemm_shared_b_equals_replicated(M, N, L, K):
    """B as one shared read-only copy gives the same bits as a replica per
    partition."""
    say(f"gemm shared B {M}x{N}x{L} K={K}")
    A, B = inputs.gemm_inputs(M, N, L, seed=M + K)
    assert np.array_equal(_gemm_dev(A, B, K, whole=jacc.SHARED), _gemm_dev(A, B, K))


@pytest.mark.parametrize("M,N,L", [(1, 1, 1), (17, 1, 9), (1, 2, 8), (33, 31, 7), (64, 63, 16), (65, 129, 71),
                                   (97, 40, 515), (513, 517, 24), (700, 1100, 40)])
def test_gemm_tiles_edges_boxes_and_nonfinite_rows(M, N, L):
    """Shapes around the wave tiles (16x32 to 64x64), the 8-deep stages and
    the 16-byte pairs (odd rows, one column): the product against the oracle
    (exact for integer inputs), a box whose edges cut pairs and tiles leaves
    the rest of C alone and has the same bits as the whole product, and an
    infinity in A's last row and a NaN in B's last column reach only that row
    and column."""
    say(f"gemm tiles {M}x{N}x{L}")
    Ai, Bi = inputs.gemm_inputs(M, N, L, seed=M + L, integer=True)
    assert np.array_equal(_gemm_dev(Ai, Bi, 1), oracle.gemm(Ai, Bi))
    A, B = inputs.gemm_inputs(M, N, L, seed=M + N)
    full = _gemm_dev(A, B, 1)
    assert np.linalg.norm(full - oracle.gemm(A, B)) <= 1e-12 * np.linalg.norm(A) * np.linalg.norm(B)
    for r0, r1, c0, c1 in ((0, M, N - 1, N), (M // 3, M, N // 2, N), (0, (M + 1) // 2, N // 3, max(N // 3, N - 1))):
        C = np.full((M, N), 7.0)
        want = C.copy()
        want[r0:r1, c0:c1] = full[r0:r1, c0:c1]
        with context(1) as c:
            c.enter(A)
            c.enter(B, whole=True)
            c.enter(C)
            c.loop(jacc.GEMM, jacc.bounds((r0, r1), (c0, c1)),
                   [(A, jacc.READ, 0, 0, 0), (B, jacc.READ, 0, 0, 1), (C, jacc.WRITE, 0, 0, 0)])
            c.exit(C)
        assert np.array_equal(C, want), (r0, r1, c0, c1)
    A[-1, -1], B[0, -1] = np.inf, np.nan
    got = _gemm_dev(A, B, 1)
    assert np.array_equal(got[:-1, :-1], full[:-1, :-1])
    assert not np.isfinite(got[-1]).any() and np.isnan(got[:, -1]).all()


def _rows_matrix(lens, ncols, seed):
    """CSR matrix with the given row lengths, columns uniform with
    replacement (unsorted, duplicates kept), values N(0,1)."""
    r = np.random.default_rng(seed)
    rp = np.zeros(len(lens) + 1, dtype=np.int32)
    np.cumsum(lens, out=rp[1:])
    col = r.integers(0, ncols, size=int(rp[-1])).astype(np.int32)
    return rp, col, r.standard_normal(int(rp[-1])), r.random(ncols) * 2 - 1


@pytest.mark.parametrize("case,ncols", [("empty_rows", 16384), ("long_rows", 16385), ("dense_block", 40000),
                                        ("short_rows", 300000), ("one_row", 70000), ("wide", (2048 << 14) + 5)])
def test_binned_spmv_edges(case, ncols):
    """The binned form where its blocks end: column counts around the
    16384-column blocks and past the 2048 blocks whose counters fit LDS in the
    build, empty rows, rows longer than a row block holds, a run of dense
    rows (whose row blocks are summed from the CSR arrays) whose place in the
    partitions differs with K, unsorted columns and duplicates.  Every row
    within the bound, and the same bits for K = 1, 4 and 20."""
    say(f"binned spmv {case} {ncols} columns")
    r = np.random.default_rng(len(case))
    n = 1 if case == "one_row" else 3001
    lens = {"empty_rows": r.integers(0, 3, n) * r.integers(0, 2, n), "long_rows": r.integers(0, 700, n),
            "dense_block": np.where((np.arange(n) > 700) & (np.arange(n) < 760), 9000, 3),
            "short_rows": r.integers(0, 5, n), "one_row": np.array([30000]), "wide": r.integers(0, 40, n)}[case]
    rp, col, val, x = _rows_matrix(lens, ncols, seed=31)
    ref = oracle.spmv_csr(rp, col, val, x)
    bound = 1e-13 * _row_bound(rp, col, val, x)
    cfg = jacc.config(order=4)
    ys = [_spmv_dev(rp, col, val, x, K, cfg) for K in (1, 4, 20) if K <= n]
    assert np.all(np.abs(ys[0] - ref) <= bound)
    for y in ys[1:]:
        assert np.array_equal(y, ys[0])


def test_binned_products_of_one_matrix_on_two_streams():
    """Two independent products of one matrix land on different streams and
    share its device copy: each waits for the other's use of the copy."""
    say("binned products on two streams")
    n = 200_000
    rp, col, val, x1 = inputs.csr_matrix(n, n, 16, seed=33)
    x2 = inputs.uniform(n, seed=34, lo=-1.0, hi=1.0)
    y1, y2 = np.zeros(n), np.zeros(n)
    cfg = jacc.config(order=4)
    with context(2) as c:
        c.enter(rp, halo=(1, 1), K=1)
        for a in (col, val, x1, x2):
            c.enter(a, whole=True, K=1)
        for y in (y1, y2):
            c.enter(y, clause=jacc.CREATE, K=1)
        for _ in range(30):
            c.spmv(rp, col, val, x1, y1, cfg=cfg)
            c.spmv(rp, col, val, x2, y2, cfg=cfg)
        c.exit(y1)
        c.exit(y2)
    for x, y in ((x1, y1), (x2, y2)):
        ref = oracle.spmv_csr(rp, col, val, x)
        assert np.all(np.abs(y - ref) <= 1e-13 * _row_bound(rp, col, val, x))


@pytest.mark.parametrize("lanes,per_row", [(4, 3), (8, 7), (16, 13)])
def test_plain_spmv_lanes_follow_the_mean_row_length(lanes, per_row):
    say(f"spmv default lanes for {per_row} entries a row")
    rp, col, val, x = _rows_matrix(np.full(5003, per_row), 5003, seed=per_row)
    y = _spmv_dev(rp, col, val, x, 1)
    assert np.array_equal(y, _spmv_dev(rp, col, val, x, 1, jacc.config(tile=lanes, order=2)))
    assert np.array_equal(y, _spmv_dev(rp, col, val, x, 3))
    assert np.all(np.abs(y - oracle.spmv_csr(rp, col, val, x)) <= 1e-13 * _row_bound(rp, col, val, x))


@pytest.mark.parametrize("flags", [0, jacc.INIT_NO_PACK])
def test_banded_matrix_with_a_halo_x(flags):
    """2^20 rows of up to 5 neighbours with x entered with a halo: every
    partition reads its own slab, so a second product after x changed by a
    loop of the partitions is that of the new x (by default and with order 4,
    K = 1 and 4)."""
    say(f"banded matrix, halo x, flags={flags}")
    n = (1 << 20) + 3
    cols = np.arange(n)[:, None] + np.arange(-2, 3)[None, :]
    keep = (cols >= 0) & (cols < n)
    rp = np.concatenate([[0], np.cumsum(keep.sum(axis=1))]).astype(np.int32)
    col = cols[keep].astype(np.int32)
    val = inputs.uniform(col.size, seed=41, lo=-1.0, hi=1.0)
    x0 = inputs.uniform(n, seed=42, lo=-1.0, hi=1.0)
    ref1 = oracle.spmv_csr(rp, col, val, x0)
    ref2 = oracle.spmv_csr(rp, col, val, ref1)
    bound1 = 1e-13 * _row_bound(rp, col, val, x0)
    # the second product's error carries the first's through |A|
    bound2 = 1e-13 * _row_bound(rp, col, val, ref1) + oracle.spmv_csr(rp, col, np.abs(val), bound1)
    for K in (1, 4):
        for cfg in (None, jacc.config(order=4)):
            x, y = x0.copy(), np.zeros(n)
            with context(K, flags) as c:
                c.enter(rp, halo=(1, 1))
                for a in (col, val):
                    c.enter(a, whole=True)
                c.enter(x, halo=(2, 2))
                c.enter(y, halo=(2, 2), clause=jacc.CREATE)
                for src, dst in ((x, y), (y, x)):
                    c.loop(jacc.SPMV_CSR, jacc.bounds((0, n)),
                           [(rp, jacc.READ, 0, 1, 0), (col, jacc.READ, 0, 0, 1), (val, jacc.READ, 0, 0, 1),
                            (src, jacc.READ, -2, 2, 0), (dst, jacc.WRITE, 0, 0, 0)], cfg=cfg)
                c.exit(y)
                c.exit(x)
            assert np.all(np.abs(y - ref1) <= bound1), K
            assert np.all(np.abs(x - ref2) <= bound2), K


@pytest.mark.parametrize("timed", [False, True])
def test_binned_copy_follows_values_written_by_a_graph(timed):
    """A graph that writes the matrix's values is replayed between products:
    each product is that of the values the replay left (launched, and timed
    without a warm-up launch)."""
    say(f"binned copy and graph replays timed={timed}")
    n = 3000
    rp, col, val, x = inputs.csr_matrix(n, n, 8, seed=51)
    src = inputs.uniform(val.size, seed=52, lo=-1.0, hi=1.0)
    idx = np.arange(val.size, dtype=np.int32)
    y = np.zeros(n)
    cfg = jacc.config(order=4)
    with context(1) as c:
        for a in (rp, col, val, x, src, idx):
            c.enter(a, whole=a is src or a is idx)
        c.enter(y, clause=jacc.CREATE)
        c.batch_begin()
        c.scatter_sq(src, idx, val)
        g = c.batch_end()
        c.spmv(rp, col, val, x, y, cfg=cfg)
        for step in range(3):
            src[:] = inputs.uniform(val.size, seed=60 + step, lo=-1.0, hi=1.0)
            c.update(src, jacc.UPDATE_DEVICE)
            c.batch_time(g, warmup=0, reps=1) if timed else c.batch_launch(g)
            c.spmv(rp, col, val, x, y, cfg=cfg)
            c.update(y, jacc.UPDATE_HOST)
            now = oracle.scatter_sq(src, idx, val.copy())
            ref = oracle.spmv_csr(rp, col, now, x)
            assert np.all(np.abs(y - ref) <= 1e-13 * _row_bound(rp, col, now, x)), step
        c.exit(y)


class _NoCopyMemory(jacc.TorchAllocator):
    """PyTorch memory, refused while `refuse` is set."""
    refuse = False

    def _alloc(self, nbytes, user):
        return None if self.refuse else super()._alloc(nbytes, user)


@pytest.mark.parametrize("K", [1, 4])
@pytest.mark.parametrize("case", ["no_memory", "long_mean_row"])
def test_binned_product_falls_back_to_the_plain_form(case, K):
    """Without memory for the copy, and for a mean row longer than a row block
    holds, order 4 runs the plain form: its bits, and no error left behind."""
    say(f"binned fallback {case} K={K}")
    n, d = (4000, 12) if case == "no_memory" else (9, 11000)
    rp, col, val, x = _rows_matrix(np.full(n, d), 20000, seed=71)
    ys = []
    for cfg in (jacc.config(order=2), jacc.config(order=4)):
        mem = _NoCopyMemory()
        y = np.zeros(n)
        with jacc.Context(K, streams="torch", allocator=mem) as c:
            c.enter(rp, halo=(1, 1))
            for a in (col, val, x):
                c.enter(a, whole=True)
            c.enter(y, clause=jacc.CREATE)
            mem.refuse = case == "no_memory"
            for _ in range(2):
                c.spmv(rp, col, val, x, y, cfg=cfg)
            assert c.last_error() == ""
            mem.refuse = False
            c.exit(y)
        ys.append(y)
    assert np.array_equal(ys[0], ys[1])
    assert np.all(np.abs(ys[0] - oracle.spmv_csr(rp, col, val, x)) <= 1e-13 * _row_bound(rp, col, val, x))


@pytest.mark.parametrize("K", [1, 3])
def test_binned_products_of_boxes_and_a_changed_row_ptr(K):
    """Boxes of rows of one matrix (more of them than copies are kept) and a
    row_ptr that gives a box more and fewer entries: each product is that of
    the box's rows now, and rows outside it keep their values."""
    say(f"binned boxes K={K}")
    n = 6000
    r = np.random.default_rng(5)
    lens = [r.integers(0, 9, n), r.integers(0, 9, n), r.integers(0, 9, n)]
    lens[1][n // 2:] = 0
    lens[1][:n // 2] = 9
    lens[1][n // 2] = 1
    nnz = max(int(x.sum()) for x in lens)
    rp = np.zeros(n + 1, np.int32)
    col = r.integers(0, n, nnz).astype(np.int32)
    val, x = r.standard_normal(nnz), r.random(n)
    cfg = jacc.config(order=4)
    boxes = [(k * 1000, k * 1000 + 3000) for k in range(4)] + [(0, n), (17, 18), (2500, 2500)]
    with context(K) as c:
        c.enter(rp, halo=(1, 1))
        for a in (col, val, x):
            c.enter(a, whole=True)
        y = np.zeros(n)
        c.enter(y)
        for ls in lens:
            np.cumsum(ls, out=rp[1:])
            c.update(rp, jacc.UPDATE_DEVICE)
            ref = oracle.spmv_csr(rp, col, val, x)
            bound = 1e-13 * _row_bound(rp, col, val, x)
            for lo, hi in boxes + boxes[::-1]:
                y[:] = 7.0
                c.update(y, jacc.UPDATE_DEVICE)
                c.loop(jacc.SPMV_CSR, jacc.bounds((lo, hi)),
                       [(rp, jacc.READ, 0, 1, 0), (col, jacc.READ, 0, 0, 1), (val, jacc.READ, 0, 0, 1),
                        (x, jacc.READ, 0, 0, 1), (y, jacc.WRITE, 0, 0, 0)], cfg=cfg)
                c.update(y, jacc.UPDATE_HOST)
                assert np.all(np.abs(y[lo:hi] - ref[lo:hi]) <= bound[lo:hi]), (lo, hi)
                assert np.all(y[:lo] == 7.0) and np.all(y[hi:] == 7.0)
        c.exit(y)


@pytest.mark.parametrize("mean,lanes", [(2, 4), (4, 8), (7, 16), (15, 16)])
def test_binned_rows_beyond_lds(mean, lanes):
    """Rows on both sides of the longest that a lane group adds (8192 entries)
    and of the 16384 products a workgroup holds at a time, some in blocks of
    other long rows, the rest short: the plain form's bits with the same lanes,
    for K = 1, 4 and 20, and every row within the bound."""
    say(f"binned rows beyond LDS, mean {mean}")
    n = 60000
    lens = np.random.default_rng(mean).integers(0, 2 * mean, n)
    lens[:6] = (8191, 8192, 8193, 1, 9000, 0)
    lens[30000:30005] = (16383, 16384, 16385, 40001, 2000)
    lens[-1] = 9601
    rp, col, val, x = _rows_matrix(lens, 50000, seed=mean)
    plain = _spmv_dev(rp, col, val, x, 1, jacc.config(tile=lanes, order=2))
    assert np.all(np.abs(plain - oracle.spmv_csr(rp, col, val, x)) <= 1e-13 * _row_bound(rp, col, val, x))
    for K in (1, 4, 20):
        assert np.array_equal(_spmv_dev(rp, col, val, x, K, jacc.config(order=4)), plain), K


@pytest.mark.parametrize("ncols", [20000, 200 << 14])
def test_binned_buckets_of_any_size(ncols):
    """One row block whose entries lie in one column block but for a few: bucket
    sizes around what the 16 or 64 lanes of a bucket take at once, and around
    those that a wave and the whole workgroup take; then all rows of a banded
    matrix.  The plain form's bits."""
    say(f"binned bucket sizes, {ncols} columns")
    r = np.random.default_rng(7)
    for size in (31, 32, 33, 63, 64, 65, 66, 127, 129, 255, 256, 257, 1023, 1024, 1025, 1026, 2049, 7001):
        lens = np.bincount(r.integers(0, 64, size + 3), minlength=64)
        rp, col, val, x = _rows_matrix(lens, ncols, seed=size)
        col[:] = r.integers(0, 16384, col.size)
        col[r.permutation(col.size)[:3]] = ncols - 1
        plain = _spmv_dev(rp, col, val, x, 1, jacc.config(order=2))
        assert np.array_equal(_spmv_dev(rp, col, val, x, 1, jacc.config(order=4)), plain), size
        assert np.all(np.abs(plain - oracle.spmv_csr(rp, col, val, x)) <= 1e-13 * _row_bound(rp, col, val, x)), size
    n = 19999
    rp, col, val, x = _rows_matrix(np.full(n, 5), ncols, seed=3)
    col[:] = (np.arange(n)[:, None] * (ncols // n) + np.array([-300, -1, 0, 1, 300])).ravel() % ncols
    plain = _spmv_dev(rp, col, val, x, 1, jacc.config(order=2))
    for K in (1, 4):
        assert np.array_equal(_spmv_dev(rp, col, val, x, K, jacc.config(order=4)), plain), K


@pytest.mark.parametrize("rows,ncols", [(1003, (1 << 21) + 7), (5, 1 << 20), (70001, (1 << 20) + 1)])
def test_sparse_matrix_with_many_columns(rows, ncols):
    """Matrices that the default leaves to the plain form for their few entries
    a column: one launch over the partitions, a launch each, and both forms give
    the same bits (K = 1, 4 and 16)."""
    say(f"spmv {rows} rows, {ncols} columns")
    lens = np.random.default_rng(rows).integers(0, 30, rows)
    rp, col, val, x = _rows_matrix(lens, ncols, seed=rows)
    ref = _spmv_dev(rp, col, val, x, 1, jacc.config(order=2))
    assert np.all(np.abs(ref - oracle.spmv_csr(rp, col, val, x)) <= 1e-13 * _row_bound(rp, col, val, x))
    for K in (k for k in (1, 4, 16) if k <= rows):
        for cfg in (None, jacc.config(order=4)):
            assert np.array_equal(_spmv_dev(rp, col, val, x, K, cfg), ref), (K, cfg)


@pytest.mark.parametrize("M,N,L", [(3, 3, 1 << 22), (17, 40, (1 << 22) + 5), (5, (1 << 25) + 3, 3), (33, 1 << 25, 2),
                                   (65, (1 << 25) + 1, 2)])
def test_gemm_beyond_32_bit_offsets(M, N, L):
    """Rows of A from 2^22 elements and rows of B from 2^25 (a lane's offsets
    take 64 bits), for each of the tiles that such shapes take: exact for
    integer inputs."""
    say(f"gemm {M}x{N}x{L}")
    r = np.random.default_rng(M)
    A = r.integers(-8, 9, (M, L)).astype(np.float64)
    B = r.integers(-8, 9, (L, N), dtype=np.int8).astype(np.float64)
    C = _gemm_dev(A, B, 1, whole=jacc.SHARED)
    say("  product done")
    for c0 in range(0, N, 1 << 22):
        assert np.array_equal(C[:, c0:c0 + (1 << 22)], A @ B[:, c0:c0 + (1 << 22)])


def test_gemm_of_more_rows_than_a_launch_has_tiles_for():
    """2^29 and more rows of one column: their 32-row tiles are more workgroups
    than one launch takes."""
    m = (1 << 29) + 77
    say(f"gemm {m}x1x1")
    A = np.arange(m, dtype=np.float64).reshape(m, 1)
    C = _gemm_dev(A, np.array([[3.0]]), 1)
    assert np.array_equal(C, 3.0 * A)


@pytest.mark.parametrize("lanes", [4, 8, 16])
def test_plain_spmv_long_rows_have_the_same_bits_alone_and_among_others(lanes):
    """A row on both sides of the length from which a wave works out a row's
    products together (2048) and of its chunks of 512: alone in a wave, where
    that is done, and in a wave of such rows, where each has its own lanes."""
    say(f"plain spmv, long rows, {lanes} lanes")
    for length in (2047, 2048, 2049, 2559, 2560, 2561, 4100, 30001):
        rp, col, val, x = _rows_matrix(np.array([length]), 5000, seed=length)
        bound = 1e-13 * _row_bound(rp, col, val, x)[0]
        want = oracle.spmv_csr(rp, col, val, x)[0]
        got = []
        for many in (False, True):
            lens = np.full(200, length if many else 3)
            lens[100] = length
            rp2 = np.zeros(201, np.int32)
            np.cumsum(lens, out=rp2[1:])
            col2, val2 = np.tile(col, 200)[:rp2[-1]].copy(), np.tile(val, 200)[:rp2[-1]].copy()
            col2[rp2[100]:rp2[101]], val2[rp2[100]:rp2[101]] = col, val
            for K in (1, 3):
                got.append(_spmv_dev(rp2, col2, val2, x, K, jacc.config(tile=lanes, order=2))[100])
        assert abs(got[0] - want) <= bound and all(g == got[0] for g in got), length
