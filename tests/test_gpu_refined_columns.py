"""Refinement of several columns: the one launch (k_fg_rest) and separate
launches take the columns in lockstep through the same side-by-side triangles,
so every column's iterate is the same bit for bit, whichever way the iterations
run: rows over more than eight lanes, dense blocks, restarts, a second group,
columns that stop early.

kkt_update_matrix with the factored values makes a handle launch every
iteration of its budget separately; without it, iterations that nothing
announced run in the one launch.  eta_target = 0 makes every iteration of the
budget run (a zero column stops after the direct solve).
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


@pytest.mark.parametrize("op", ["N", "T"])
@pytest.mark.parametrize("B,nrhs,zero,opts", [
    (40, 2, (), dict(fgmres_max_iters=3, solve_entries_per_lane=1)),  # rows over many lanes
    (300, 8, (0, 7), dict(fgmres_max_iters=2, solve_entries_per_lane=1, solve_chain=4)),
    (500, 5, (2,), dict(fgmres_max_iters=3, dense_tail=100)),         # dense block, padded
    (20, 3, (), dict(fgmres_max_iters=2, dense_tail=196)),            # the whole matrix dense
    (200, 11, (9,), dict(fgmres_max_iters=5, fgmres_restart=2, dense_tail=33, matching=1)),
    (2000, 3, (), dict(fgmres_max_iters=2)),
    (100, 4, (1,), dict(fgmres_max_iters=3, debug_schedule=1)),       # adversarial tickets
])
def test_columns_bitwise(B, nrhs, zero, opts, op):
    pat, seq = kktgen.make_sequence(B, 78, 2, nrhs)
    vals, b = dev(seq[1][0]), seq[1][1].reshape(nrhs, pat.n).copy()
    b[list(zero)] = 0.0
    out = []
    for separate in (False, True):
        s = binding.KKTSolver(eta_target=0.0, **opts)
        s.analyze(pat.n, pat.rowptr, pat.colind, seq[0][0])
        s.refactor(vals)
        if separate:
            s.update_matrix(vals)
        x = s.solve(dev(b.ravel()), op=op).cpu().numpy()
        out.append((x.reshape(nrhs, pat.n), s.report()))
        s.close()
    (x1, r1), (x2, r2) = out
    assert r1.iters == r2.iters == opts["fgmres_max_iters"]
    assert r1.eta == r2.eta <= 1e-12
    for c in range(nrhs):
        assert np.array_equal(x1[c].view(np.int64), x2[c].view(np.int64)), c
    assert not x1[list(zero)].any()
