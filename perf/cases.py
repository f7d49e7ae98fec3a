"""The work this runtime is used for, as cases to be timed.

A case is a dict of plain values.  ``listed()`` names the ones that stand for
the uses below, ``draw(rng)`` gives another of the same ranges, ``prepare``
makes what a program holds before the call (arrays entered into a context,
a captured graph, a model with its weights), ``run`` is one pass through the
public entry points, ``exact`` the same results from plain torch in 64 bits,
and ``work`` the bytes and operations a pass cannot do without.

Kinds and what they stand for:

* ``jacobi``: time stepping of a 2-D 5-point stencil between two arrays that
  stay on the device, from cache-resident grids whose steps cost a launch
  each to grids bound by memory; one partition or several, split by rows or
  by columns; issued step by step or replayed from a captured graph.
* ``heat``: the 3-D 7-point step with its residual reduced every step and
  read back after a few steps, as a convergence loop does.
* ``sum``: a reduction whose value the host needs before it goes on.
* ``gemm``: the dense FP64 contraction, square and ragged.
* ``spmv``: the CSR product of an iterative solver, from matrices whose x
  fits a cache to 2^22 rows.
* ``batch``: an application's many independent sweeps of uneven sizes,
  replayed as one graph (small loops as tasks of one launch).
* ``train`` and ``predict``: fitting the launch-cost network on timings, and
  evaluating it over a loop's candidate configurations.
"""
import numpy as np
import torch

from paper_2110_14340_amd import inputs, jacc

DEV = "cuda:0"
FEATURES = jacc.NFEATURES


def listed():
    return [
        # cache-resident grid, issued step by step: launch latency
        {"name": "jacobi_512", "kind": "jacobi", "ny": 512, "nx": 512, "K": 1, "part_dim": 0, "steps": 20, "graph": 0},
        # the benchmark's headline: 8192^2 over 8 row-block partitions
        {"name": "jacobi_8192_k8", "kind": "jacobi", "ny": 8192, "nx": 8192, "K": 8, "part_dim": 0, "steps": 10, "graph": 0},
        # odd extents, split by columns into 4 partitions
        {"name": "jacobi_ragged_cols", "kind": "jacobi", "ny": 4099, "nx": 3001, "K": 4, "part_dim": 1, "steps": 10, "graph": 0},
        # a captured time-stepping loop over 4 partitions, each step one task launch
        {"name": "jacobi_512_k4_graph", "kind": "jacobi", "ny": 512, "nx": 512, "K": 4, "part_dim": 0, "steps": 20, "graph": 1},
        # 3-D field bound by memory, 4 partitions, residual every step
        {"name": "heat_512_k4", "kind": "heat", "nz": 512, "ny": 512, "nx": 512, "K": 4, "steps": 5, "residual": 1},
        # small field of odd extents, residual every step
        {"name": "heat_ragged", "kind": "heat", "nz": 95, "ny": 131, "nx": 203, "K": 1, "steps": 10, "residual": 1},
        # the benchmark's reduction, read by the host
        {"name": "sum_512c", "kind": "sum", "n": 1 << 27, "K": 1, "squares": 0},
        # the benchmark's contraction
        {"name": "gemm_4096", "kind": "gemm", "M": 4096, "N": 4096, "L": 4096, "K": 1, "shared": 0},
        # ragged contraction over 3 partitions that share B
        {"name": "gemm_ragged", "kind": "gemm", "M": 1000, "N": 777, "L": 1531, "K": 3, "shared": 1},
        # the benchmark's sparse product: 2^22 rows, 4 partitions sharing the matrix
        {"name": "spmv_2e22", "kind": "spmv", "rows": 1 << 22, "per_row": 16, "K": 4, "shared": 1},
        # 32 uneven 2-D and 3-D sweeps as one graph
        {"name": "batch_uneven", "kind": "batch", "n2d": 16, "n3d": 16, "shape_seed": 5, "side2d": 4096, "side3d": 512},
        # one epoch of the launch-cost network in minibatches of 256
        {"name": "cost_model_train", "kind": "train", "n": 2000, "batch": 256, "epochs": 1},
    ]


def _log_int(rng, lo, hi):
    return int(min(hi, lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["jacobi", "jacobi", "heat", "heat", "sum", "gemm", "spmv", "batch", "train", "predict"])
    if kind == "jacobi":
        ny, nx = _log_int(rng, 64, 8192), _log_int(rng, 64, 8192)
        part_dim = rng.choice([0, 0, 1])
        return {"kind": kind, "ny": ny, "nx": nx, "K": rng.choice([1, 2, 4, 8]), "part_dim": part_dim,
                "steps": 10 if ny * nx > 1 << 22 else 20, "graph": 0 if part_dim else rng.choice([0, 0, 1])}
    if kind == "heat":
        z, y, x = (_log_int(rng, 24, 512) for _ in range(3))
        return {"kind": kind, "nz": z, "ny": y, "nx": x, "K": rng.choice([1, 2, 4]), "steps": 5,
                "residual": rng.choice([0, 1, 1])}
    if kind == "sum":
        return {"kind": kind, "n": _log_int(rng, 1000, 1 << 26), "K": rng.choice([1, 2, 4]), "squares": rng.choice([0, 1])}
    if kind == "gemm":
        return {"kind": kind, "M": _log_int(rng, 32, 4096), "N": _log_int(rng, 32, 4096), "L": _log_int(rng, 32, 4096),
                "K": rng.choice([1, 2, 4]), "shared": rng.choice([0, 1])}
    if kind == "spmv":
        return {"kind": kind, "rows": _log_int(rng, 1000, 1 << 22), "per_row": rng.randint(4, 16),
                "K": rng.choice([1, 2, 4]), "shared": rng.choice([0, 1])}
    if kind == "batch":
        return {"kind": kind, "n2d": rng.randint(2, 16), "n3d": rng.randint(2, 16), "shape_seed": rng.randrange(1000),
                "side2d": 2048, "side3d": 256}
    if kind == "train":
        return {"kind": kind, "n": _log_int(rng, 100, 2000), "batch": rng.choice([64, 256]), "epochs": 1}
    return {"kind": kind, "n": _log_int(rng, 30, 20000)}


# ---- inputs: from the seed alone, made on the device, held by the host ---------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _uniform(g, *shape, lo=0.0, hi=1.0):
    return torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64).mul_(hi - lo).add_(lo)


def _grid(case, g):
    """Interior uniform[0,1), boundary 0 (the distribution of inputs.jacobi_grid)."""
    u = _uniform(g, case["ny"], case["nx"])
    u[0], u[-1], u[:, 0], u[:, -1] = 0.0, 0.0, 0.0, 0.0
    return u


def _csr(case, g):
    """Column draws uniform with replacement, sorted, duplicates dropped (the
    recipe of inputs.csr_matrix): (row_ptr, col, val, x)."""
    n, d = case["rows"], case["per_row"]
    cols = torch.randint(0, n, (n, d), generator=g, device=DEV, dtype=torch.int32).sort(dim=1).values
    keep = torch.ones_like(cols, dtype=torch.bool)
    keep[:, 1:] = cols[:, 1:] != cols[:, :-1]
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rp[1:] = keep.sum(dim=1).cumsum(0)
    col = cols[keep]
    val = torch.randn(col.numel(), generator=g, device=DEV, dtype=torch.float64)
    return rp.to(torch.int32), col, val, _uniform(g, n, lo=-1.0, hi=1.0)


def _shapes(case):
    return inputs.batch_shapes(case["shape_seed"], case["n2d"], case["n3d"], side2d=(64, case["side2d"]),
                               side3d=(32, case["side3d"]))


def _fields(case, g):
    return [_grid({"ny": s[0], "nx": s[1]}, g) if len(s) == 2 else _uniform(g, *s) for s in _shapes(case)]


def _samples(n, g):
    """Features, targets (a smooth function of them) and initial weights."""
    X = torch.randn(n, FEATURES, generator=g, device=DEV, dtype=torch.float64).float()
    w = torch.randn(FEATURES, generator=g, device=DEV, dtype=torch.float64)
    y = torch.nn.functional.softplus(X.double() @ w * 0.5).float()
    W = inputs.mlp_init(FEATURES, seed=int(torch.randint(1 << 30, (1,), generator=g, device=DEV)))
    return X.cpu().numpy(), y.cpu().numpy(), {k: v.astype(np.float32) for k, v in W.items()}


# ---- state -------------------------------------------------------------------
class _State:
    """What a program holds between calls; closes its context when dropped."""

    def __init__(self, K):
        self.ctx, self.model = jacc.Context(K), None

    def __del__(self):
        if self.model is not None:
            self.model.close()
        self.ctx.close()


def _owned(ctx, a, K, part_dim=0):
    """The device blocks that partitions 0..K-1 own of entered array `a`."""
    out = []
    E = a.shape[part_dim]
    for p in range(K):
        dev, lo, hi = ctx.slab(a, p)
        own = slice(p * E // K, (p + 1) * E // K)
        buf = ctx.allocator.live[dev].view(torch.float64)
        if part_dim == 0:
            out.append(buf.view(hi - lo, *a.shape[1:])[own.start - lo:own.stop - lo])
        else:  # a column slab: from an even column, with an even pitch
            base = lo & ~1
            out.append(buf.view(a.shape[0], (hi - base + 1) & ~1)[:, own.start - base:own.stop - base])
    return out


def prepare(case, seed):
    kind, g = case["kind"], _gen(seed)
    s = _State(case.get("K", 1))
    s.case, c = case, s.ctx
    if kind in ("jacobi", "heat"):
        u = _grid(case, g) if kind == "jacobi" else _uniform(g, case["nz"], case["ny"], case["nx"])
        s.a = u.cpu().numpy()
        s.b = s.a.copy()
        pd = case.get("part_dim", 0)
        c.enter(s.a, halo=(1, 1), part_dim=pd)
        c.enter(s.b, halo=(1, 1), part_dim=pd)
        last = s.a if case["steps"] % 2 == 0 else s.b
        s.out = _owned(c, last, case["K"], pd)
        if case.get("graph"):
            cfg = jacc.config(persistent=1)
            c.batch_begin()
            for t in range(case["steps"]):
                c.jacobi2d(*((s.a, s.b) if t % 2 == 0 else (s.b, s.a)), cfg=cfg)
            s.graph = c.batch_end()  # the captured steps take effect once here
    elif kind == "sum":
        s.a = _uniform(g, case["n"], lo=-1.0).cpu().numpy()
        c.enter(s.a)
    elif kind == "gemm":
        s.A = _uniform(g, case["M"], case["L"], lo=-1.0).cpu().numpy()
        s.B = _uniform(g, case["L"], case["N"], lo=-1.0).cpu().numpy()
        s.C = np.zeros((case["M"], case["N"]))
        c.enter(s.A)
        c.enter(s.B, whole=jacc.SHARED if case["shared"] else True)
        c.enter(s.C, clause=jacc.CREATE)
        s.out = _owned(c, s.C, case["K"])
    elif kind == "spmv":
        s.csr = [t.cpu().numpy() for t in _csr(case, g)]
        s.y = np.zeros(case["rows"])
        c.enter(s.csr[0], halo=(1, 1))
        for a in s.csr[1:]:
            c.enter(a, whole=jacc.SHARED if case["shared"] else True)
        c.enter(s.y, clause=jacc.CREATE)
        s.out = _owned(c, s.y, case["K"])
    elif kind == "batch":
        s.ins = [u.cpu().numpy() for u in _fields(case, g)]
        s.outs = [u.copy() for u in s.ins]
        s.out = []
        for u, v in zip(s.ins, s.outs):
            c.enter(u, halo=(1, 1))
            c.enter(v, halo=(1, 1))
            s.out += _owned(c, v, 1)
        c.batch_begin()
        for u, v in zip(s.ins, s.outs):
            cfg = jacc.config(persistent=1) if u.size < 1 << 18 else None
            if u.ndim == 2:
                c.jacobi2d(u, v, cfg=cfg)
            else:
                c.heat3d(u, v, 0.1, cfg=cfg)
        s.graph = c.batch_end()
    else:
        s.X, s.t, W = _samples(case["n"], g)
        s.model = jacc.Model(c, FEATURES)
        s.model.set_params(W)
    return s


def run(s):
    case, c = s.case, s.ctx
    kind = case["kind"]
    if kind == "jacobi":
        if case["graph"]:
            c.batch_launch(s.graph)
        else:
            for t in range(case["steps"]):
                if t % 2 == 0:
                    c.jacobi2d(s.a, s.b)
                else:
                    c.jacobi2d(s.b, s.a)
        return s.out
    if kind == "heat":
        for t in range(case["steps"]):
            u, v = (s.a, s.b) if t % 2 == 0 else (s.b, s.a)
            c.heat3d(u, v, 0.1, slot=t if case["residual"] else -1)
        return {"field": s.out, "residuals": c.reductions(0, case["steps"]) if case["residual"] else None}
    if kind == "sum":
        return c.sum(s.a, squares=bool(case["squares"]))
    if kind == "gemm":
        c.gemm(s.A, s.B, s.C)
        return s.out
    if kind == "spmv":
        c.spmv(*s.csr, s.y)
        return s.out
    if kind == "batch":
        c.batch_launch(s.graph)
        return s.out
    if kind == "train":
        losses = s.model.train(s.X, s.t, epochs=case["epochs"], batch=case["batch"], lr=1e-3, seed=7)
        return {"losses": losses, "weights": s.model.pack(s.model.get_params())}
    return s.model.predict(s.X)


# ---- the same from plain torch in 64 bits -------------------------------------
def _jacobi_step(u):
    v = u.clone()
    v[1:-1, 1:-1] = 0.25 * ((u[:-2, 1:-1] + u[2:, 1:-1]) + (u[1:-1, :-2] + u[1:-1, 2:]))
    return v


def _heat_step(u):
    v, c = u.clone(), u[1:-1, 1:-1, 1:-1]
    lap = u[1:-1, 1:-1, :-2] + u[1:-1, 1:-1, 2:]
    lap += u[1:-1, :-2, 1:-1] + u[1:-1, 2:, 1:-1]
    lap += u[:-2, 1:-1, 1:-1] + u[2:, 1:-1, 1:-1]
    lap -= 6.0 * c
    v[1:-1, 1:-1, 1:-1] += 0.1 * lap
    return v, float((v - u).square_().sum())


def _blocks(u, K, dim=0):
    E = u.shape[dim]
    return [u.narrow(dim, p * E // K, (p + 1) * E // K - p * E // K) for p in range(K)]


def _forward(W, X):
    h = [X]
    for k in "123":
        h.append(torch.relu(h[-1] @ W["W" + k].T + W["b" + k]))
    return h, h[3] @ W["w4"] + W["b4"]


def _order(n, state):
    """The shuffled sample order of the next epoch: Fisher-Yates with
    splitmix64 numbers, as training documents it."""
    perm, mask = list(range(n)), (1 << 64) - 1
    for i in range(n - 1, 0, -1):
        state = (state + 0x9E3779B97F4A7C15) & mask
        z = ((state ^ (state >> 30)) * 0xBF58476D1CE4E5B9) & mask
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & mask
        j = (z ^ (z >> 31)) % (i + 1)
        perm[i], perm[j] = perm[j], perm[i]
    return perm, state


def _train(X, t, W, batch, epochs, lr=1e-3, seed=7):
    n, step, state, losses = len(t), 0, seed, []
    bsz = min(batch, n)
    m = {k: torch.zeros_like(v) for k, v in W.items()}
    v2 = {k: torch.zeros_like(v) for k, v in W.items()}
    for _ in range(epochs):
        perm, state = _order(n, state)
        total = 0.0
        for o in range(0, n, bsz):
            idx = torch.tensor(perm[o:o + bsz], device=X.device)
            h, y = _forward(W, X[idx])
            e = y - t[idx]
            total += float(e.square().sum())
            g = 2.0 * e / len(idx)
            grad = {"w4": g @ h[3], "b4": g.sum().reshape(1)}
            d = g[:, None] * W["w4"] * (h[3] > 0)
            for k in (3, 2, 1):
                grad["W%d" % k], grad["b%d" % k] = d.T @ h[k - 1], d.sum(0)
                if k > 1:
                    d = (d @ W["W%d" % k]) * (h[k - 1] > 0)
            step += 1
            for k in W:
                m[k] = 0.9 * m[k] + 0.1 * grad[k]
                v2[k] = 0.999 * v2[k] + 0.001 * grad[k].square()
                W[k] = W[k] - lr * (m[k] / (1 - 0.9 ** step)) / ((v2[k] / (1 - 0.999 ** step)).sqrt() + 1e-8)
        losses.append(total / n)
    return np.array(losses), W


def exact(case, seed):
    kind, g = case["kind"], _gen(seed)
    if kind == "jacobi":
        u = _grid(case, g)
        for _ in range(case["steps"] * (2 if case["graph"] else 1)):  # a capture takes effect once
            u = _jacobi_step(u)
        return _blocks(u, case["K"], case["part_dim"])
    if kind == "heat":
        u, res = _uniform(g, case["nz"], case["ny"], case["nx"]), []
        for _ in range(case["steps"]):
            u, r = _heat_step(u)
            res.append(r)
        return {"field": _blocks(u, case["K"]), "residuals": np.array(res) if case["residual"] else None}
    if kind == "sum":
        x = _uniform(g, case["n"], lo=-1.0)
        return float((x * x if case["squares"] else x).sum())
    if kind == "gemm":
        A = _uniform(g, case["M"], case["L"], lo=-1.0)
        return _blocks(A @ _uniform(g, case["L"], case["N"], lo=-1.0), case["K"])
    if kind == "spmv":
        rp, col, val, x = _csr(case, g)
        rows = torch.repeat_interleave(torch.arange(case["rows"], device=DEV), (rp[1:] - rp[:-1]).long())
        y = torch.zeros(case["rows"], dtype=torch.float64, device=DEV)
        return _blocks(y.index_add_(0, rows, val * x[col.long()]), case["K"])
    if kind == "batch":
        return [_jacobi_step(u) if u.ndim == 2 else _heat_step(u)[0] for u in _fields(case, g)]
    X, t, W = _samples(case["n"], g)
    X, t = torch.from_numpy(X).double().to(DEV), torch.from_numpy(t).double().to(DEV)
    W = {k: torch.from_numpy(v).double().to(DEV) for k, v in W.items()}
    if kind == "train":
        losses, W = _train(X, t, W, case["batch"], case["epochs"])
        return {"losses": losses, "weights": torch.cat([W[k].reshape(-1) for k in jacc.PARAM_ORDER])}
    return _forward(W, X)[1]


def work(case):
    kind = case["kind"]
    if kind in ("jacobi", "heat"):
        dims = [case["ny"], case["nx"]] + ([case["nz"]] if kind == "heat" else [])
        cells = float(np.prod([max(0, d - 2) for d in dims])) * case["steps"]
        return {"bytes": 16.0 * cells, "flops": (4.0 if kind == "jacobi" else 9.0) * cells}
    if kind == "sum":
        return {"bytes": 8.0 * case["n"], "flops": (2.0 if case["squares"] else 1.0) * case["n"]}
    if kind == "gemm":
        M, N, L = case["M"], case["N"], case["L"]
        return {"bytes": 8.0 * (M * L + L * N + M * N), "flops": 2.0 * M * N * L}
    if kind == "spmv":
        n = case["rows"]
        nnz = n * n * (1.0 - (1.0 - 1.0 / n) ** case["per_row"])  # expected distinct columns
        return {"bytes": 4.0 * (n + 1) + 12.0 * nnz + 16.0 * n, "flops": 2.0 * nnz}
    if kind == "batch":
        cells = sum(float(np.prod([d - 2 for d in s])) for s in _shapes(case))
        return {"bytes": 16.0 * cells, "flops": 9.0 * cells}
    weights = 64 * FEATURES + 2 * 64 * 64 + 4 * 64 + 1
    n = case["n"] * case.get("epochs", 1)
    if kind == "train":
        return {"bytes": 4.0 * ((FEATURES + 1) * n + 2 * weights), "flops": 6.0 * weights * n}
    return {"bytes": 4.0 * ((FEATURES + 1) * n + weights), "flops": 2.0 * weights * n}
