"""Batch validation: one entry that leaves its graph, at the edges of the graphs' entry ranges."""
from __future__ import annotations

import numpy as np
import pytest

import graphgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sizes", [[1], [300, 0, 1, 5_000], [2] * 9_000, [70_001, 3]])
def test_crossing_entry_is_found(sizes):
    import paper_2204_05821_amd as kb
    gs = []
    for i, n in enumerate(sizes):
        m = 3 * n if i % 3 else n
        src, dst = graphgen.uniform_edges(n, m, i + 1) if n else (np.zeros(0, np.int32), np.zeros(0, np.int32))
        gs.append(graphgen.from_edges(n, src, dst, None, None))
    rp, col, el, vl, vp, off = kb.union_of(gs)
    dev = lambda a: None if a is None else torch.from_numpy(a).cuda()
    b = kb.Batch(dev(rp), dev(col), dev(el), dev(vl), dev(vp), off, kmax=2)
    ids, counts = b.refine(2)
    b.close()
    for g in range(0, len(sizes), max(1, len(sizes) // 8)):
        if gs[g].m == 0:
            continue
        r = kb.refiner_for(gs[g], kmax=2)
        one, cnt = r.refine(2)
        assert cnt == counts[g]
        for x, y in zip(one, ids):
            assert torch.equal(x, y[off[g]:off[g + 1]])
        r.close()
    ends = [g for g in range(len(sizes)) if gs[g].m]
    for g in (ends[0], ends[-1]):
        for e in (rp[off[g]], rp[off[g + 1]] - 1):
            for bad in (off[g] - 1, off[g + 1]):
                if not 0 <= bad < off[-1]:
                    continue
                c2 = col.copy()
                c2[e] = bad
                with pytest.raises(kb.KbisimError) as ei:
                    kb.Batch(dev(rp), dev(c2), dev(el), dev(vl), dev(vp), off, kmax=2)
                assert ei.value.code == kb.EGRAPH
