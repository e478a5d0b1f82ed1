"""Short-row kernel at the edges of its layouts: factors bit for bit against
the oracle (an fma per update in ascending pivot order, so there is nothing to
tolerate).

A banded matrix makes every row one run: row i has min(i, w) pivots and up to
2 w + 1 entries, so w = 31, 32, 63, 64, 127 put rows at 63, 65, 127, 129 and
255 entries, on both sides of a 64-position word, of the one-, two- and
four-word forms, and at the kernel's limit of 256; its pivots pass 64, the size
of a diagonal batch.  Runs are cut at the workgroup's waves (8 for systems that
fit the chip at once, 4 in a large batch) and start anew at a row that does not
depend on the one before it.  Arrow matrices give rows that are no run at all.
"""
import numpy as np
import pytest

import oracle
from paper_2306_14337_amd import binding

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.lib()
    yield


def csr(mask, seed):
    """Diagonally dominant values on the pattern, natural pivots."""
    rng = np.random.default_rng(seed)
    n = mask.shape[0]
    np.fill_diagonal(mask, True)
    r, c = np.nonzero(mask)
    v = rng.standard_normal(len(r))
    v[r == c] += 4.0 * n
    rp = np.zeros(n + 1, np.int64)
    np.add.at(rp, r + 1, 1)
    return n, np.cumsum(rp), c.astype(np.int32), v


def banded(n, w, starts=()):
    """Banded blocks; row d in starts opens a block (it does not depend on the
    row before it)."""
    i = np.arange(n)
    m = np.abs(i[:, None] - i[None, :]) <= w
    for d in starts:
        m[d:, :d] = m[:d, d:] = False
    return m


def check(n, rp, ci, v0, new, count=1, **opts):
    s = binding.KKTSolver(ordering=1, **opts)
    if count > 1:
        s.analyze_shared(n, rp, ci, v0, count)
    else:
        s.analyze(n, rp, ci, v0)
    s.refactor(torch.from_numpy(np.concatenate(new)).to("cuda:0"))
    lu = s.lu()[2].reshape(count, -1)
    rep = s.report()
    assert rep.min_pivot > 0.0
    o = oracle.OracleLU(n, rp, ci, v0, Q=np.arange(n), tau=1e-10)
    for t in range(0, count, max(1, count - 1)):
        o.refactor(new[t])
        f = o.factors()
        rows = np.concatenate([f["Li"], f["Ui"]])
        cols = np.concatenate([np.repeat(np.arange(n), np.diff(f["Lp"])),
                               np.repeat(np.arange(n), np.diff(f["Up"]))])
        want = np.concatenate([f["Lx"], f["Ux"]])[np.lexsort((cols, rows))]
        assert np.array_equal(lu[t].view(np.int64), want.view(np.int64)), t


def values(v, seed, count=1):
    rng = np.random.default_rng(seed)
    return [v * (1.0 + 0.1 * rng.standard_normal(v.size)) for _ in range(count)]


@pytest.mark.parametrize("w", [1, 4, 31, 32, 63, 64, 127])
def test_banded_runs(w):
    n, rp, ci, v = csr(banded(2 * w + 40, w), w)
    check(n, rp, ci, v, values(v, 1), dense_tail=-1)


@pytest.mark.parametrize("w", [3, 32, 70])
def test_cut_runs(w):
    m = banded(200, w, starts=(3, 4, 9, 17, 64, 65, 128))
    n, rp, ci, v = csr(m, w)
    check(n, rp, ci, v, values(v, 2), dense_tail=-1)


def test_no_runs():
    m = np.zeros((150, 150), bool)
    m[140:, :] = m[:, 140:] = True  # ten dense rows and columns: long rows, dense end
    n, rp, ci, v = csr(m, 5)
    check(n, rp, ci, v, values(v, 3), dense_tail=-1)


@pytest.mark.parametrize("count", [2, 60])
def test_shared_batch_packs_runs(count):
    """2 instances fit the chip at once (runs of 8), 60 x 150 rows do not (4)."""
    n, rp, ci, v = csr(banded(150, 33, starts=(20, 51)), 7)
    check(n, rp, ci, v, values(v, 4, count), count=count)
