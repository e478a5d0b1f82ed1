"""Long-row kernel at the edges of its units: factors bit for bit against the
oracle (an fma per update in ascending pivot order, so there is nothing to
tolerate).

Bands of 128 to 520 rows put every row behind the first ones in one chain of
runs, whose pivots have 128 to 521 columns: pieces of 64 with and without a
remainder, one and two units of the pivots inside a run (256 columns) and of the
row before it (512).  Dense blocks of 1 to 20 rows with a dense border give the
border's rows pivot blocks of every size up to 8, with columns behind them that
end on both sides of a piece.  A workgroup stages eight rows of up to 2,400
entries, four of up to 4,800, else one: arrows of 2,000, 2,500 and 5,000 rows.
"""
import numpy as np
import pytest

from paper_2306_14337_amd import binding
from test_gpu_short_rows import banded, check, csr, values

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.lib()
    yield


def blocks(sizes, border):
    n = sum(sizes) + border
    m = np.zeros((n, n), bool)
    d = 0
    for s in sizes:
        m[d:d + s, d:d + s] = True
        d += s
    m[d:, :] = m[:, d:] = True
    return m


@pytest.mark.parametrize("w", [128, 129, 192, 255, 256, 511, 512, 520])
def test_band(w):
    n, rp, ci, v = csr(banded(w + 300, w), w)
    check(n, rp, ci, v, values(v, w), dense_tail=-1)


@pytest.mark.parametrize("border", [3, 52, 63, 64, 120, 140])
def test_pivot_blocks(border):
    sizes = [1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 16, 20] * 4
    n, rp, ci, v = csr(blocks(sizes, border), border)
    check(n, rp, ci, v, values(v, border), dense_tail=-1)


@pytest.mark.parametrize("count", [2, 5])
def test_instances(count):
    n, rp, ci, v = csr(blocks([9, 4, 1, 17] * 6, 70), count)
    check(n, rp, ci, v, values(v, count, count), count=count, dense_tail=-1)


@pytest.mark.parametrize("n", [2000, 2500, 5000])
def test_staging(n):
    n, rp, ci, v = csr(blocks([1, 8, 2] * ((n - 14) // 11), 14), n)
    check(n, rp, ci, v, values(v, n), dense_tail=-1)
