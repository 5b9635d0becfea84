"""Device transpose, by sorting and entry by entry, against the host transpose."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

import graphgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _rows(n, rp, col, el):
    """Entries (row, label, column) in a canonical order."""
    row = np.repeat(np.arange(n), np.diff(rp))
    lab = np.zeros(len(col), np.int64) if el is None else el
    at = np.lexsort((lab, col, row))
    return np.stack([row, np.asarray(lab)[at], np.asarray(col)[at]])


# sorted from 2^20 entries on: whole and ragged chunks of 2048; rows per chunk past the marked limit
# (8192), most of them empty; one hub target; labels so wide that the sort key does not fit
M = 1 << 20
CASES = [(1, 1, 1), (300, 2049, 0), (1, M, 0), (2, M + 1, 3), (70_001, M - 1, 40), (70_001, M + 2047, 40),
         (5_000_011, M + 2049, 3), (100_003, M, 1 << 31), (1_000_003, M, 0)]


@pytest.mark.parametrize("n,m,labels", CASES)
@pytest.mark.parametrize("hub", [False, True])
@pytest.mark.parametrize("small_workspace", [False, True])
def test_transpose(n, m, labels, hub, small_workspace):
    import paper_2204_05821_amd as kb
    print(f"[transpose] n={n} m={m} labels={labels} hub={hub} small={small_workspace}", flush=True)
    rng = np.random.default_rng(m)
    src, dst = rng.integers(0, n, m), rng.integers(0, n, m)
    if hub:
        src[: m // 2] = n // 2
        dst[m // 3:] = n - 1
    lab = rng.integers(0, labels, m).astype(np.int32) if labels else None
    g = graphgen.from_edges(n, src, dst, lab)
    rp, col, el, _, _ = kb.to_device(g)
    if small_workspace:
        lib = kb._lib()
        size = ctypes.c_size_t(0)
        assert lib.kbisim_transpose_workspace_bytes(n, 0, ctypes.byref(size)) == 0
        ws = torch.empty(size.value, dtype=torch.uint8, device="cuda")
        trp, tcol = torch.empty_like(rp), torch.empty_like(col)
        tel = None if el is None else torch.empty_like(el)
        p = kb._ptr
        torch.cuda.synchronize()
        assert lib.kbisim_transpose(n, m, p(rp), p(col), p(el), p(trp), p(tcol), p(tel), p(ws), size.value, None) == 0
    else:
        trp, tcol, tel = kb.transpose(rp, col, el)
    h = graphgen.transpose(g)
    assert np.array_equal(trp.cpu().numpy(), h.row_ptr)
    got = _rows(n, h.row_ptr, tcol.cpu().numpy(), None if tel is None else tel.cpu().numpy())
    assert np.array_equal(got, _rows(n, h.row_ptr, h.col, h.elabel))
