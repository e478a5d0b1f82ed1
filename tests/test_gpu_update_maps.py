"""Rows of the short-row band that go by masks keep no update positions: the
device memory of a handle whose rows are all short stays below that of one
whose rows all have map entries, but for the masks."""
import numpy as np
import pytest

from paper_2306_14337_amd import binding, kktgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,micro", [(300, 0), (300, -1), (1000, 0)])
def test_masks_in_place_of_map_entries(B, micro):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pat, seq = kktgen.make_sequence(B, 5, 1)
    size = {}
    for short in (0, -1):
        s = binding.KKTSolver(refactor_short_rows=short, refactor_long_rows=-1,
                              refactor_micro_rows=micro, dense_tail=-1)
        s.analyze(pat.n, pat.rowptr, pat.colind, seq[0][0])
        info = s.info()
        size[short] = info.device_bytes
        rp, ci, _ = s.lu()
        s.close()
    length = np.diff(rp)
    assert length.max() <= 256
    row = np.repeat(np.arange(pat.n), length)
    pivots = np.bincount(row[ci < row], minlength=pat.n)
    masks = 8 * int((pivots * np.where(length <= 64, 1, np.where(length <= 128, 2, 4))).sum())
    upper = length - pivots - 1  # U entries behind the diagonal
    adds = int(upper[ci[ci < row]].sum())
    # micro rows (at most 8 entries) keep at most 4 map entries each; row
    # metadata (16 bytes), flags and chunk tables: at most 64 bytes a row
    kept = 2 * 4 * int((length <= 8).sum()) if micro == 0 else 0
    assert size[0] - size[-1] <= masks - 2 * adds + kept + 64 * pat.n
    assert 2 * adds > 64 * pat.n  # the map is more than what the bound leaves open
