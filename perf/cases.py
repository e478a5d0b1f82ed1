"""Workloads of the solver, as a user's program runs them through the binding.

The users are interior-point and scenario codes: one analysis per grid, then
many systems of that grid's pattern.  Every case is one pass of such a loop on
inputs that are already on the GPU:

  step     refactor(values) and solve(b) of the next interior-point system
  solve    more right-hand sides for factors that are already there (predictor
           and corrector steps, sensitivities), plain or transposed
  adjoint  a differentiable solve, forward and backward (KKTSolveFn)
  shared   a captured batch: scenarios of one grid, one analysis
  own      a captured batch: grids of different sizes, block-diagonal
  refine   a step with a fixed number of refinement iterations

All arithmetic is float64, the library's only type.  The grids are the seeded
synthetic ones of ``kktgen`` (10 rows per bus); the sizes go from its smallest
to its largest grid in use, 100 to 70,000 buses.
"""
import functools
import math

import numpy as np
import torch

from paper_2306_14337_amd import binding, kktgen

DEV = "cuda:0"
GRID = 101  # seed of a case's grid; a case's own seed draws the systems on it

# buses -> nonzeros of the factors per nonzero of A, multiply-adds of the
# factorization per row, of the host analysis on these grids
_FILL_B = np.log([100, 300, 1000, 3000, 10000, 25000, 70000])
_FILL = [1.42, 1.49, 1.54, 1.59, 1.73, 1.81, 1.99]
_MADDS = [55.0, 66.0, 79.0, 94.0, 161.0, 223.0, 479.0]


def listed():
    return [
        # The smallest grid: a feeder or a teaching network, where a step is all
        # latency and launches; library defaults.
        dict(name="step_100", kind="step", buses=100, nrhs=1, budget=0),
        # A regional grid of ordinary size, library defaults.
        dict(name="step_1000", kind="step", buses=1000, nrhs=1, budget=0),
        # A national grid, an odd size, library defaults.
        dict(name="step_9973", kind="step", buses=9973, nrhs=1, budget=0),
        # The headline sequence: the largest grid with the adaptive launch
        # budget, as the benchmark runs it.
        dict(name="step_70000", kind="step", buses=70000, nrhs=1, budget=-1),
        # A corrector step on a large grid: one more right-hand side for the
        # factors of the last step.
        dict(name="solve_30000", kind="solve", buses=30000, nrhs=1, op="N", budget=-1),
        # Sensitivities of a regional grid: a handful of transposed solves.
        dict(name="solve_t_3001", kind="solve", buses=3001, nrhs=5, op="T", budget=0),
        # One training step through a small grid's solution.
        dict(name="adjoint_500", kind="adjoint", buses=500, nrhs=1, budget=0),
        # The adjoint workload: 32 right-hand sides forward and backward.
        dict(name="adjoint_10000", kind="adjoint", buses=10000, nrhs=32, budget=-1),
        # Contingency screening on a small grid, in one captured graph.
        dict(name="shared_64x500", kind="shared", buses=500, count=64, budget=0),
        # The batched workload's shared group: 128 scenarios of 2,000 buses.
        dict(name="shared_128x2000", kind="shared", buses=2000, count=128, budget=0),
        # The batched workload's uneven group: grids of 500 to 5,000 buses.
        dict(name="own_32", kind="own", buses=5000, count=32, budget=0),
        # Fixed-step refinement: two forced iterations after the direct solve.
        dict(name="refine_10000", kind="refine", buses=10000, nrhs=1, iters=2, budget=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "solve", "adjoint", "shared", "own", "refine"])
    c = dict(kind=kind, budget=rng.choice([0, -1]))
    if kind == "step":
        c.update(buses=_log_int(rng, 100, 70000), nrhs=1)
    elif kind == "solve":
        c.update(buses=_log_int(rng, 300, 30000), nrhs=rng.randint(1, 6), op=rng.choice("NT"))
    elif kind == "adjoint":
        nrhs = _log_int(rng, 1, 32)
        c.update(buses=_log_int(rng, 200, 10000), nrhs=nrhs)
    elif kind == "shared":
        buses = _log_int(rng, 200, 2000)
        c.update(buses=buses, count=_log_int(rng, 4, min(256, 256000 // buses)), budget=0)
    elif kind == "own":
        c.update(buses=_log_int(rng, 1000, 5000), count=rng.randint(4, 32), budget=0)
    else:
        c.update(buses=_log_int(rng, 300, 20000), nrhs=1, iters=rng.randint(1, 3), budget=0)
    return c


@functools.lru_cache(maxsize=96)
def _grid(buses, seed):
    return kktgen.make_kkt(buses, seed)


def _grids(case):
    """The grids of a case: one, or one per instance of an uneven batch."""
    if case["kind"] != "own":
        return [_grid(case["buses"], GRID)]
    hi = case["buses"]
    sizes = np.random.default_rng(GRID).integers(max(100, hi // 10), hi + 1, size=case["count"])
    return [_grid(int(b), GRID * 1000 + i) for i, b in enumerate(sizes)]


def _inputs(case, seed):
    """Host inputs from the seed: per grid the first system's values (for the
    analysis), then the systems of the pass (instances back to back), the
    right-hand sides and, for the adjoint, the cotangents."""
    rng = np.random.default_rng([GRID, seed])
    grids = _grids(case)
    first = [g.values(kktgen.draw_sigma(rng, g.n_p)) for g in grids]
    inst = grids * case["count"] if case["kind"] == "shared" else grids
    vals = np.concatenate([g.values(kktgen.draw_sigma(rng, g.n_p)) for g in inst])
    b = rng.standard_normal(sum(g.n for g in inst) * case.get("nrhs", 1))
    c = rng.standard_normal(b.size) if case["kind"] == "adjoint" else None
    return grids, inst, first, vals, b, c


def prepare(case, seed):
    kind = case["kind"]
    grids, inst, first, vals, b, c = _inputs(case, seed)
    opts = dict(refine_budget=case["budget"])
    if kind == "refine":
        opts["min_iters"] = case["iters"]
    s = binding.KKTSolver(**opts)
    g = grids[0]
    if kind == "shared":
        s.analyze_shared(g.n, g.rowptr, g.colind, first[0], case["count"])
    elif kind == "own":
        s.analyze_batch([(p.n, p.rowptr, p.colind, v) for p, v in zip(grids, first)],
                        list(range(len(grids))))
    else:
        s.analyze(g.n, g.rowptr, g.colind, first[0])
    st = dict(kind=kind, solver=s, op=case.get("op", "N"), values=torch.from_numpy(vals).to(DEV),
              b=torch.from_numpy(b).to(DEV))
    st["x"] = torch.zeros_like(st["b"])
    if kind == "adjoint":
        st["c"] = torch.from_numpy(c).to(DEV)
        st["values"].requires_grad_(True)
        st["b"].requires_grad_(True)
    elif kind == "solve":
        s.refactor(st["values"])
    elif kind in ("shared", "own"):
        st["stream"] = torch.cuda.Stream()
        torch.cuda.synchronize()
        s.graph_capture(st["values"], st["b"], st["x"], st["stream"])
    return st


def run(state):
    s, kind = state["solver"], state["kind"]
    if kind in ("step", "refine"):
        s.refactor(state["values"])
        return s.solve(state["b"], state["x"])
    if kind == "solve":
        return s.solve(state["b"], state["x"], op=state["op"])
    if kind == "adjoint":
        x = binding.KKTSolveFn.apply(s, state["values"], state["b"])
        gv, gb = torch.autograd.grad(x, (state["values"], state["b"]), state["c"])
        return dict(x=x.detach(), grad_values=gv, grad_b=gb)
    s.graph_launch(torch.cuda.current_stream())
    return state["x"]


def work(case):
    """Values and right-hand sides read, solutions (and gradients) written,
    index structures and factors touched once; the factorization's and the
    solves' multiply-adds."""
    kind, nrhs = case["kind"], case.get("nrhs", 1)
    by = fl = 0.0
    grids = _grids(case)
    for g in grids:
        at = math.log(max(100, g.B))
        count = case["count"] if kind == "shared" else 1
        f = g.nnz * float(np.interp(at, _FILL_B, _FILL))
        madds = g.n * float(np.interp(at, _FILL_B, _MADDS))
        index = 4 * g.nnz + 4 * f + 8 * g.n
        solves = nrhs * (case.get("iters", 0) + 1 + (kind == "adjoint"))
        by += index
        if kind == "solve":
            by += 8 * (f + g.nnz) + 16 * g.n * nrhs
        else:
            by += count * (8 * g.nnz + 8 * f + 16 * g.n * nrhs)
            fl += count * 2 * madds
        if kind == "adjoint":
            by += 8 * g.nnz + 16 * g.n * nrhs
            fl += 2 * g.nnz * nrhs
        fl += count * solves * 2 * (f + g.nnz)
    return {"bytes": by, "flops": fl}


def _dense_solver(g, vals):
    """Solves with A and its transpose: a dense LU of the symmetrically
    equilibrated matrix and one correction with the residual in long double."""
    rows = np.repeat(np.arange(g.n), np.diff(g.rowptr))
    cols = g.colind.astype(np.int64)
    dev = DEV if torch.cuda.is_available() else "cpu"
    big = np.zeros(g.n)
    np.maximum.at(big, rows, np.abs(vals))
    d = 2.0 ** -np.round(0.5 * np.log2(big))
    A = torch.zeros((g.n, g.n), dtype=torch.float64, device=dev)
    A[torch.from_numpy(rows).to(dev), torch.from_numpy(cols).to(dev)] = \
        torch.from_numpy(vals * d[rows] * d[cols]).to(dev)
    lu, piv = torch.linalg.lu_factor(A)
    del A
    order = np.argsort(cols, kind="stable")
    starts = {False: g.rowptr[:-1], True: np.concatenate([[0], np.cumsum(np.bincount(cols, minlength=g.n))])[:-1]}
    src = {False: cols, True: rows[order]}
    long_vals = {False: vals.astype(np.longdouble), True: vals[order].astype(np.longdouble)}

    def apply(r, t):
        y = torch.from_numpy(np.asarray(r * d, dtype=np.float64)).to(dev).unsqueeze(1)
        return torch.linalg.lu_solve(lu, piv, y, adjoint=t).squeeze(1).cpu().numpy() * d

    def solve(b, t=False):
        x = np.zeros(g.n, dtype=np.longdouble)
        for _ in range(3):
            ax = np.add.reduceat(long_vals[t] * x[src[t]], starts[t])
            x = x + apply(b - ax, t)
        return x.astype(np.float64)

    return solve


def exact(case, seed):
    """The solutions and gradients from dense factorizations, for grids and
    batches that a dense factorization takes within seconds."""
    kind, nrhs = case["kind"], case.get("nrhs", 1)
    grids, inst, _, vals, b, c = _inputs(case, seed)
    if sum(float(g.n) ** 3 for g in inst) > 1.0e12:
        return None
    xs, at, row = [], 0, 0
    for g in inst:
        v = vals[at:at + g.nnz]
        solve = _dense_solver(g, v)
        bs = b[row:row + g.n * nrhs].reshape(nrhs, g.n)
        xs.append(np.concatenate([solve(r, case.get("op") == "T") for r in bs]))
        at, row = at + g.nnz, row + g.n * nrhs
    x = np.concatenate(xs)
    if kind != "adjoint":
        return torch.from_numpy(x)
    g = grids[0]
    lam = np.concatenate([solve(r, True) for r in c.reshape(nrhs, g.n)])
    rows = np.repeat(np.arange(g.n), np.diff(g.rowptr))
    X, L = x.reshape(nrhs, g.n), lam.reshape(nrhs, g.n)
    gv = -sum(L[k][rows] * X[k][g.colind] for k in range(nrhs))
    return dict(x=torch.from_numpy(x), grad_values=torch.from_numpy(gv), grad_b=torch.from_numpy(lam))
