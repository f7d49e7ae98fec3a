"""GPU parity of batched execution: captured single-stream hipGraphs of
partitioned loop sequences, replayed several times with eager work and host
reads between replays, and persistent-kernel task groups of many small
uneven sweeps — every output bit-identical to the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_2110_14340_amd import inputs, jacc
from gpu_util import context, say

pytestmark = pytest.mark.gpu


def test_graph_of_two_jacobi_steps_replayed_with_eager_work_between():
    say("graph replay jacobi 130x98 K=4")
    u0 = inputs.jacobi_grid(130, 98, seed=21)
    a, b = u0.copy(), u0.copy()
    with context(4) as c:
        c.enter(a, halo=(1, 1))
        c.enter(b, halo=(1, 1))
        c.jacobi2d(a, b)
        c.jacobi2d(b, a)
        c.batch_begin()
        c.jacobi2d(a, b)
        c.jacobi2d(b, a)
        g = c.batch_end()          # runs once: 4 steps so far
        assert c.batch_info(g)["replay_safe"]
        steps = 4
        for r in range(4):
            c.batch_launch(g, 1 + r)
            steps += 2 * (1 + r)
            c.update(a, jacc.UPDATE_HOST)
            assert np.array_equal(a, oracle.jacobi2d(u0, steps)), f"replay {r}"
            if r % 2 == 0:         # eager work between replays
                c.jacobi2d(a, b)
                c.jacobi2d(b, a)
                steps += 2
        c.exit(b)
        c.exit(a)
    assert np.array_equal(a, oracle.jacobi2d(u0, steps))


def test_graph_of_heat_steps_with_residual_slots():
    say("graph replay heat 30x20x36 K=2 with residuals")
    u0 = inputs.heat_field(30, 20, 36, seed=22)
    a, b = u0.copy(), u0.copy()
    with context(2) as c:
        c.enter(a, halo=(1, 1))
        c.enter(b, halo=(1, 1))
        c.heat3d(a, b, 0.1, slot=10)   # eager steps first: the captured pair is then a fixed point
        c.heat3d(b, a, 0.1, slot=11)
        c.batch_begin()
        c.heat3d(a, b, 0.1, slot=0)
        c.heat3d(b, a, 0.1, slot=1)
        g = c.batch_end()
        assert c.batch_info(g)["replay_safe"]
        r01 = c.reductions(0, 2)
        c.batch_launch(g, 1)
        r23 = c.reductions(0, 2)
        c.exit(a)
        c.exit(b)
    ref, ref_res = oracle.heat3d(u0, 6, 0.1)
    assert np.array_equal(a, ref)
    assert np.all(np.abs(r01 - ref_res[2:4]) <= 1e-13 * ref_res[2:4])
    assert np.all(np.abs(r23 - ref_res[4:6]) <= 1e-13 * ref_res[4:6])


def _batch_members(seed, n2, n3):
    r = np.random.default_rng(seed)
    shapes = [(int(r.integers(3, 90)), int(r.integers(3, 700))) for _ in range(n2)]
    shapes += [(int(r.integers(3, 20)), int(r.integers(3, 20)), int(r.integers(3, 300))) for _ in range(n3)]
    return shapes


def test_persistent_group_of_uneven_sweeps_bit_exact():
    say("persistent group: 24 uneven 2-D/3-D sweeps")
    shapes = _batch_members(23, 16, 8)
    cfgs = [jacc.config(tile=t, vec=v, persistent=1, march=m) for t in (1, 3, 8) for v in (1, 2) for m in (1, 2)]
    ins, outs, refs = [], [], []
    with context(4) as c:
        for i, sh in enumerate(shapes):
            u = inputs.jacobi_grid(*sh, seed=100 + i) if len(sh) == 2 else inputs.heat_field(*sh, seed=100 + i)
            v = u.copy()
            c.enter(u, halo=(1, 1), K=1)
            c.enter(v, halo=(1, 1), K=1)
            ins.append(u)
            outs.append(v)
            ref = u.copy()
            if len(sh) == 2:
                oracle.jacobi2d_sweep(u, ref)
            else:
                oracle.heat3d_sweep(u, ref, 0.1)
            refs.append(ref)
        c.batch_begin()
        for i, sh in enumerate(shapes):
            cf = cfgs[i % len(cfgs)]
            if cf.vec == 2 and sh[-1] % 2:
                cf = jacc.config(tile=cf.tile, vec=1, persistent=1, march=cf.march)
            if len(sh) == 2:
                c.jacobi2d(ins[i], outs[i], cfg=cf)
            else:
                c.heat3d(ins[i], outs[i], 0.1, cfg=cf)
        g = c.batch_end()
        info = c.batch_info(g)
        assert info["persistent_groups"] == 1 and info["replay_safe"]
        for rep in range(3):
            c.batch_launch(g, 1)
            for i in range(len(shapes)):
                c.update(outs[i], jacc.UPDATE_HOST)
                assert np.array_equal(outs[i], refs[i]), (rep, i, shapes[i])
                outs[i][...] = -1.0   # host copy scribbled between replays
        for i in range(len(shapes)):
            c.exit(outs[i])
            c.exit(ins[i])
    for i in range(len(shapes)):
        assert np.array_equal(outs[i], refs[i])


def test_batch_mixing_persistent_and_partitioned_loops():
    say("batch: persistent small loops + K=2 large loop")
    big = inputs.jacobi_grid(300, 260, seed=31)
    small = [inputs.jacobi_grid(20 + i, 33 + 2 * i, seed=40 + i) for i in range(5)]
    with context(2) as c:
        a, b = big.copy(), big.copy()
        c.enter(a, halo=(1, 1))
        c.enter(b, halo=(1, 1))
        outs = []
        for s in small:
            o = s.copy()
            c.enter(s, halo=(1, 1), K=1)
            c.enter(o, halo=(1, 1), K=1)
            outs.append(o)
        c.jacobi2d(a, b)
        c.jacobi2d(b, a)
        c.batch_begin()
        for s, o in zip(small, outs):
            c.jacobi2d(s, o, cfg=jacc.config(tile=4, vec=1, persistent=1))
        c.jacobi2d(a, b)
        c.jacobi2d(b, a)
        g = c.batch_end()
        assert c.batch_info(g) == {"loops": 7, "persistent_groups": 1, "replay_safe": True}
        c.batch_launch(g, 2)
        for s, o in zip(small, outs):
            c.exit(o)
            c.exit(s)
        c.exit(b)
        c.exit(a)
    assert np.array_equal(a, oracle.jacobi2d(big, 8))
    for s, o in zip(small, outs):
        ref = s.copy()
        oracle.jacobi2d_sweep(s, ref)
        assert np.array_equal(o, ref)


def test_graph_of_partitioned_steps_as_persistent_tasks_k8():
    say("graph: 8 partitions per step as persistent tasks, mirrors, 20 replays")
    u0 = inputs.jacobi_grid(515, 1030, seed=51)
    a, b = u0.copy(), u0.copy()
    cfg = jacc.config(tile=8, vec=2, persistent=1)
    with context(8) as c:
        c.enter(a, halo=(1, 1))
        c.enter(b, halo=(1, 1))
        c.batch_begin()
        c.jacobi2d(a, b, cfg=cfg)
        c.jacobi2d(b, a, cfg=cfg)
        g = c.batch_end()
        assert c.batch_info(g) == {"loops": 2, "persistent_groups": 2, "replay_safe": True}
        c.batch_launch(g, 19)
        c.exit(b)
        c.exit(a)
    assert np.array_equal(a, oracle.jacobi2d(u0, 40))


@pytest.mark.parametrize("shape,K,steps", [
    ((3, 3), 1, 4), ((9, 9), 4, 5), ((40, 66), 1, 2), ((40, 66), 2, 3), ((33, 43), 3, 12), ((34, 44), 1, 13),
    ((12, 300), 5, 24), ((300, 12), 16, 23), ((130, 127), 2, 20), ((257, 200), 4, 40),
    ((2100, 1300), 3, 25), ((1500, 2200), 8, 9),  # enough regions for the tall ones
])
def test_chained_steps_bit_exact(shape, K, steps):
    """Persistent steps between two arrays whose boundaries differ, as a graph,
    replayed: both arrays afterwards, every partition's slabs included."""
    say(f"chained steps {shape} K={K} steps={steps}")
    a = inputs.jacobi_grid(*shape, seed=61)
    b = inputs.jacobi_grid(*shape, seed=62)
    for u, v in ((a, 0.25), (b, -0.75)):
        u[0], u[-1], u[:, 0], u[:, -1] = v, 2 * v, 3 * v, 4 * v
    ref = [a.copy(), b.copy()]
    cfg = jacc.config(persistent=1)
    with context(K) as c:
        c.enter(a, halo=(1, 1))
        c.enter(b, halo=(1, 1))
        c.batch_begin()
        for t in range(steps):
            c.jacobi2d(*((a, b) if t % 2 == 0 else (b, a)), cfg=cfg)
        g = c.batch_end()
        assert c.batch_info(g) == {"loops": steps, "persistent_groups": steps, "replay_safe": True}
        c.batch_launch(g, 2)
        c.jacobi2d(a, b)  # reads every partition's halo rows
        c.jacobi2d(b, a)
        c.exit(b, jacc.COPYOUT)
        c.exit(a, jacc.COPYOUT)
    for t in [t for _ in range(3) for t in range(steps)] + [0, 1]:
        oracle.jacobi2d_sweep(ref[t % 2], ref[1 - t % 2])
    assert np.array_equal(a, ref[0]) and np.array_equal(b, ref[1])


@pytest.mark.parametrize("K,box", [(1, ((5, 40), (7, 100))), (3, ((20, 61), (1, 129))), (4, ((30, 33), (60, 62)))])
def test_chained_steps_of_an_inner_box_between_other_loops(K, box):
    """A box inside the grid keeps what either array holds around it; a sum, a
    loop on other arrays and a step of another box end or join the chain."""
    say(f"chained steps box={box} K={K}")
    a, b = inputs.uniform((64, 130), seed=63), inputs.uniform((64, 130), seed=64)
    p, q = inputs.jacobi_grid(50, 70, seed=65), inputs.jacobi_grid(50, 70, seed=66)
    ref = [x.copy() for x in (a, b, p, q)]
    cfg = jacc.config(persistent=1)
    whole = ((1, 63), (1, 129))

    def sweep(u, v, bx):
        oracle.jacobi2d_sweep(u, v, bx)

    with context(K) as c:
        for x in (a, b, p, q):
            c.enter(x, halo=(1, 1))

        def step(u, v, bx):
            c.loop(jacc.JACOBI2D, jacc.bounds(*bx), [(u, jacc.READ, -1, 1, 0), (v, jacc.WRITE, 0, 0, 0)], cfg=cfg)

        c.batch_begin()
        for t in range(8):
            step(*((a, b) if t % 2 == 0 else (b, a)), box)
        step(p, q, ((1, 49), (1, 69)))            # joins the last step's group
        step(q, p, ((1, 49), (1, 69)))
        for t in range(5):
            step(*((a, b) if t % 2 == 0 else (b, a)), box)
        c.sum(a, slot=0, sync=False)              # ends the chain
        for t in range(5, 12):
            step(*((a, b) if t % 2 == 0 else (b, a)), whole if t == 8 else box)
        step(a, b, box)
        step(a, b, box)                           # not a step back
        g = c.batch_end()
        got = c.reductions(0, 1)[0]
        for x in (a, b, p, q):
            c.exit(x, jacc.COPYOUT)
    for t in range(8):
        sweep(*((ref[0], ref[1]) if t % 2 == 0 else (ref[1], ref[0])), box)
    sweep(ref[2], ref[3], ((1, 49), (1, 69)))
    sweep(ref[3], ref[2], ((1, 49), (1, 69)))
    for t in range(5):
        sweep(*((ref[0], ref[1]) if t % 2 == 0 else (ref[1], ref[0])), box)
    total = ref[0].sum()
    for t in range(5, 12):
        sweep(*((ref[0], ref[1]) if t % 2 == 0 else (ref[1], ref[0])), whole if t == 8 else box)
    sweep(ref[0], ref[1], box)
    for x, y in zip((a, b, p, q), ref):
        assert np.array_equal(x, y)
    # two sums of n values in different orders: n eps of the sum of their magnitudes
    assert abs(got - total) <= a.size * np.finfo(np.float64).eps * np.abs(ref[0]).sum() * 2


def _check_merged(shapes, K=1, replays=2, chain=False):
    """One loop per field, no configuration; with `chain` also the step back and
    a second output from the same input.  All bits as the oracle's sweeps."""
    ins = [inputs.jacobi_grid(*s, seed=200 + i) if len(s) == 2 else inputs.heat_field(*s, seed=200 + i)
           for i, s in enumerate(shapes)]
    outs, more = [u + 0.5 for u in ins], [u - 0.5 for u in ins]
    refs = [[x.copy() for x in t] for t in zip(ins, outs, more)]

    def sweep(u, v):
        oracle.jacobi2d_sweep(u, v) if u.ndim == 2 else oracle.heat3d_sweep(u, v, 0.1)

    with context(max(K, 2)) as c:
        for x in (*ins, *outs, *more):
            c.enter(x, halo=(1, 1), K=K)

        def step(u, v):
            c.jacobi2d(u, v) if u.ndim == 2 else c.heat3d(u, v, 0.1)

        c.batch_begin()
        for u, v, w in zip(ins, outs, more):
            step(u, v)
        if chain:
            for u, v, w in zip(ins, outs, more):
                step(u, w)
                step(w, u)
        g = c.batch_end()
        n = len(shapes) * (3 if chain else 1)
        assert c.batch_info(g) == {"loops": n, "persistent_groups": 0, "replay_safe": True}
        c.batch_launch(g, replays)
        for x in (*ins, *outs, *more):
            c.exit(x, jacc.COPYOUT)
    for u, v, w in refs:
        for _ in range(1 + replays):
            sweep(u, v)
            if chain:
                sweep(u, w)
                sweep(w, u)
    for i, t in enumerate(zip(ins, outs, more)):
        for x, y in zip(t, refs[i]):
            assert np.array_equal(x, y), (i, shapes[i])


@pytest.mark.parametrize("K,chain", [(1, False), (1, True), (2, True)])
def test_merged_loops_bit_exact(K, chain):
    """Independent loops that share a launch: odd and even rows, every default
    shape's edges, fields of one cell, one that is nothing but boundary."""
    say(f"merged loops K={K} chain={chain}")
    _check_merged([(3, 3), (65, 64), (64, 65), (130, 1027), (1030, 517), (9, 4100), (3, 3, 3), (9, 10, 11), (33, 34, 129),
                   (66, 67, 121), (60, 70, 260), (17, 200, 301), (82, 80, 82), (2, 40), (5, 2, 9)], K=K, chain=chain)


def test_merged_loops_beyond_the_cache_and_the_table():
    """More than 288 MB together, with a field that then runs alone as the
    streaming shape; and more loops than the table holds."""
    say("merged loops: 330 MB")
    _check_merged([(230, 240, 181), (3000, 2001), (100, 101, 102), (4, 70), (1500, 1400), (30, 31, 32)], replays=1)
    say("merged loops: 1100 small ones")
    _check_merged([(5 + i % 7, 6 + i % 66) for i in range(1100)], replays=1)
