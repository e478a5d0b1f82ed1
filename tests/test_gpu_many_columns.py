"""Several right-hand sides side by side (k_trisolve_mr8, k_tail_mw_mr8):
every column against the oracle's plain triangular solves, with the bar of the
single-column solves (1e-8 of the column's largest entry: kappa is about 1e16,
and the sums are taken in another order)."""
import numpy as np
import pytest

import oracle
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
@pytest.mark.parametrize("nrhs,B,opts", [
    (2, 100, {}),
    (7, 100, {}),
    (8, 100, dict(solve_chain=1)),            # no chains
    (9, 100, dict(dense_tail=64)),            # a second pass of one column; two dense blocks
    (3, 20, dict(dense_tail=196)),            # the whole matrix dense, padded
    (17, 40, dict(solve_entries_per_lane=1)), # rows over many lanes
    (5, 300, dict(solve_chain=8, dense_tail=33, matching=1)),
])
def test_columns_match_the_oracle(nrhs, B, opts, op):
    pat, seq = kktgen.make_sequence(B, 31, 2, nrhs)
    s = binding.KKTSolver(fgmres_max_iters=0, **opts)
    s.analyze(pat.n, pat.rowptr, pat.colind, seq[0][0])
    s.refactor(dev(seq[1][0]))
    x = s.solve(dev(seq[1][1]), op=op).cpu().numpy().reshape(nrhs, pat.n)
    assert s.report().eta <= 1e-12
    b = seq[1][1].reshape(nrhs, pat.n)
    if opts.get("matching"):
        # the oracle factors another matrix: the same columns one at a time
        want = [s.solve(dev(c), op=op).cpu().numpy() for c in b]
    else:
        o = oracle.OracleLU(pat.n, pat.rowptr, pat.colind, seq[0][0], tau=1e-10)
        o.refactor(seq[1][0])
        want = [o.apply(c, op=op) for c in b]
    for r in range(nrhs):
        assert np.abs(x[r] - want[r]).max() <= 1e-8 * np.abs(want[r]).max(), r
