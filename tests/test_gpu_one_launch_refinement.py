"""Refinement iterations in one launch (k_fg_rest) against the same iterations
as separate launches.

kkt_update_matrix with the factored values makes a handle launch every
iteration of its budget separately; without it, iterations that nothing
announced run in the one launch.  eta_target = 0 makes every iteration of the
budget run.  Single columns and batches agree bit for bit (sums are taken in
the same order); so do several columns without a dense block.  With one, the
group's dense triangle is solved by another kernel than a single column's, so
only the etas are compared.
"""
import numpy as np
import pytest

from paper_2306_14337_amd import binding, kktgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.lib()
    yield


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda:0")


def solve_both(make, nrhs, op):
    """(x, report) of the first solve by the one launch and by separate launches."""
    out = []
    for separate in (False, True):
        s, vals, b = make(nrhs)
        s.refactor(vals)
        if separate:
            s.update_matrix(vals)
        x = s.solve(b, op=op)
        out.append((x.cpu().numpy(), s.report()))
        s.close()
    return out


def single(B, seed, **opts):
    def make(nrhs):
        pat, seq = kktgen.make_sequence(B, seed, 2, nrhs)
        s = binding.KKTSolver(eta_target=0.0, **opts)
        s.analyze(pat.n, pat.rowptr, pat.colind, seq[0][0])
        return s, dev(seq[1][0]), dev(seq[1][1])

    return make


@pytest.mark.parametrize("op", ["N", "T"])
@pytest.mark.parametrize("B,nrhs,opts", [
    (20, 1, dict(fgmres_max_iters=3)),                       # fewer rows than one workgroup
    (100, 1, dict(fgmres_max_iters=7, fgmres_restart=3)),    # restarts, an odd remainder
    (1000, 1, dict(fgmres_max_iters=10)),                    # more than one group of 8 vectors
    (300, 3, dict(fgmres_max_iters=2)),                      # several columns
    (500, 1, dict(fgmres_max_iters=3, dense_tail=100)),      # dense block, padded
    (200, 1, dict(fgmres_max_iters=2, matching=1)),          # row and column scales
    (200, 1, dict(fgmres_max_iters=3, debug_schedule=1)),    # adversarial tickets
])
def test_single_system_bitwise(B, nrhs, opts, op):
    (x1, r1), (x2, r2) = solve_both(single(B, 77, **opts), nrhs, op)
    assert r1.iters == r2.iters == opts["fgmres_max_iters"]
    assert np.array_equal(x1.view(np.int64), x2.view(np.int64))
    assert r1.eta == r2.eta <= 1e-12


def test_columns_with_dense_block():
    (_, r1), (_, r2) = solve_both(single(500, 78, fgmres_max_iters=2, dense_tail=100), 5, "N")
    assert r1.iters == r2.iters == 2
    assert r1.eta <= 1e-12 and r2.eta <= 1e-12


@pytest.mark.parametrize("op", ["N", "T"])
@pytest.mark.parametrize("shared", [True, False])
def test_batches_bitwise(shared, op):
    def make(nrhs):
        rng = np.random.default_rng(9)
        s = binding.KKTSolver(eta_target=0.0, fgmres_max_iters=3)
        pats = [kktgen.make_kkt(60 if shared else 40 + 23 * i, 5 if shared else 5 + i)
                for i in range(5)]
        first = [p.values(kktgen.draw_sigma(rng, p.n_p)) for p in pats]
        if shared:
            p = pats[0]
            s.analyze_shared(p.n, p.rowptr, p.colind, first[0], len(pats))
        else:
            s.analyze_batch([(p.n, p.rowptr, p.colind, v) for p, v in zip(pats, first)],
                            list(range(len(pats))))
        vals = np.concatenate([p.values(kktgen.draw_sigma(rng, p.n_p)) for p in pats])
        return s, dev(vals), dev(rng.standard_normal(s.n))

    (x1, r1), (x2, r2) = solve_both(make, 1, op)
    assert r1.iters == r2.iters == 3
    assert np.array_equal(x1.view(np.int64), x2.view(np.int64))


def test_replayed_graph_runs_the_budget():
    """Iterations inside a captured graph, replayed with eager work between."""
    pat, seq = kktgen.make_sequence(150, 79, 4)
    s = binding.KKTSolver(eta_target=0.0, fgmres_max_iters=2)
    s.analyze(pat.n, pat.rowptr, pat.colind, seq[0][0])
    vals, b = dev(seq[1][0]), dev(seq[1][1])
    x = torch.zeros_like(b)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    s.graph_capture(vals, b, x, stream)
    for v, r in seq[1:]:
        vals.copy_(dev(v))
        b.copy_(dev(r))
        torch.cuda.synchronize()
        s.graph_launch(stream)
        stream.synchronize()
        rep = s.report()
        got = x.clone()
        s2 = binding.KKTSolver(eta_target=0.0, fgmres_max_iters=2)
        s2.analyze(pat.n, pat.rowptr, pat.colind, seq[0][0])
        s2.refactor(vals)
        want = s2.solve(b)
        assert rep.iters == 2
        assert torch.equal(got.view(torch.int64), want.view(torch.int64))
