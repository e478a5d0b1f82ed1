"""Dense block, several columns (k_tail_mw_mr8): the diagonal's quotients are
correctly rounded divisions, also where a pivot's reciprocal overflows.

The matrix is a small coupled block and, behind it, rows with a diagonal entry
alone, all of it taken as the dense block: there the solution is b / d in one
rounding, and 0 / d is 0 for a subnormal d.
"""
import numpy as np
import pytest

from paper_2306_14337_amd import binding

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
@pytest.mark.parametrize("n,nrhs", [(40, 2), (64, 8), (97, 11)])
def test_quotients_of_the_diagonal(n, nrhs, op):
    m, sub = 6, 20  # coupled rows; a row with a subnormal pivot
    rng = np.random.default_rng(n)
    d = rng.uniform(0.1, 10.0, n) * rng.choice([-1.0, 1.0], n)
    d[sub] = 1e-310
    rowptr, col, val = [0], [], []
    for i in range(n):
        cols = range(m) if i < m else [i]
        col += cols
        val += [d[i] + 20.0 * (i < m) if j == i else rng.standard_normal() for j in cols]
        rowptr.append(len(col))
    s = binding.KKTSolver(ordering=1, dense_tail=n, fgmres_max_iters=0)
    s.analyze(n, np.array(rowptr, np.int64), np.array(col, np.int32), np.array(val))
    assert s.info().dense_tail == n
    b = rng.standard_normal((nrhs, n))
    b[:, sub] = 0.0
    x = s.solve(dev(b.ravel()), op=op).cpu().numpy().reshape(nrhs, n)
    assert np.isfinite(x).all()
    assert np.array_equal(x[:, m:], b[:, m:] / d[m:])
    A = np.zeros((n, n))
    for i in range(n):
        A[i, col[rowptr[i]:rowptr[i + 1]]] = val[rowptr[i]:rowptr[i + 1]]
    M = (A if op == "N" else A.T)[:m, :m]
    assert np.allclose(x[:, :m], np.linalg.solve(M, b[:, :m].T).T, rtol=1e-12, atol=0)
