"""Workspace of the device transpose: what it needs does not grow with the entries, what sorting
them takes is asked for separately, and without room for it they are scattered."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

import graphgen

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [0, 1, 70_001, (1 << 31) - 1])
@pytest.mark.parametrize("m", [0, (1 << 20) - 1, 1 << 20, 1 << 31, (1 << 31) + 1])
def test_sizes(n, m):
    import paper_2204_05821_amd as kb
    lib = kb._lib()

    def size(f, entries):
        out = ctypes.c_size_t(0)
        assert f(n, entries, ctypes.byref(out)) == 0
        return out.value

    need, sort = size(lib.kbisim_transpose_workspace_bytes, m), size(lib.kbisim_transpose_sort_bytes, m)
    assert need == size(lib.kbisim_transpose_workspace_bytes, 0)
    if n and 1 << 20 <= m <= 1 << 31:
        assert need + 16 * m < sort < need + 17 * m
    else:
        assert sort == need


def test_errors():
    import paper_2204_05821_amd as kb
    out = ctypes.c_size_t(0)
    for f in (kb._lib().kbisim_transpose_workspace_bytes, kb._lib().kbisim_transpose_sort_bytes):
        assert f(100, 50, None) == -1
        assert f(-1, 0, ctypes.byref(out)) == -1 and f(1, -1, ctypes.byref(out)) == -1
        assert f(1 << 31, 0, ctypes.byref(out)) == -5


@pytest.mark.gpu
@pytest.mark.parametrize("labels", [0, 5])
def test_no_room_for_sort_keys(labels, monkeypatch):
    import paper_2204_05821_amd as kb
    n, m = 70_001, (1 << 20) + 5
    rng = np.random.default_rng(labels)
    g = graphgen.from_edges(n, rng.integers(0, n, m), rng.integers(0, n, m),
                            rng.integers(0, labels, m) if labels else None)
    rp, col, el, _, _ = kb.to_device(g)
    empty, refused = torch.empty, []

    def full(*shape, **kw):
        if kw.get("dtype") is torch.uint8 and shape[0] > 16 * m:
            refused.append(shape[0])
            raise torch.cuda.OutOfMemoryError("no room")
        return empty(*shape, **kw)

    monkeypatch.setattr(torch, "empty", full)
    trp, tcol, tel = kb.transpose(rp, col, el)
    monkeypatch.undo()
    assert len(refused) == 1
    h = graphgen.transpose(g)
    assert np.array_equal(trp.cpu().numpy(), h.row_ptr)
    rows = np.repeat(np.arange(n), np.diff(h.row_ptr))

    def entries(c, lab):
        lab = np.zeros(m, np.int64) if lab is None else lab
        return np.stack([rows, c, lab])[:, np.lexsort((lab, c, rows))]

    assert np.array_equal(entries(tcol.cpu().numpy(), None if tel is None else tel.cpu().numpy()),
                          entries(h.col, h.elabel))
