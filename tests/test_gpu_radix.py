"""Device radix sort at the edges of its tiles (8192 keys, tiles dealt to 8 XCDs)."""
from __future__ import annotations

import numpy as np
import pytest

import graphgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m", [1, 8191, 8192, 8193, 7 * 8192 + 1, 8 * 8192, 9 * 8192 + 5])
@pytest.mark.parametrize("labels", [0, 300])
def test_summary_triples(m, labels):
    """Distinct (source id, label, target id) triples against numpy's unique."""
    import paper_2204_05821_amd as kb
    n = 5_003
    print(f"[radix] m={m} labels={labels}", flush=True)
    src, dst = graphgen.uniform_edges(n, m, 11)
    lab = graphgen.edge_labels(m, labels, 0.0, 11) if labels else None
    g = graphgen.from_edges(n, src, dst, lab, None, name="radix")
    rng = np.random.default_rng(m)
    a, b = (rng.integers(0, n, size=n).astype(np.int32) // 7 for _ in range(2))
    r = kb.refiner_for(g, kmax=1)
    got = torch.stack(r.quotient(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()), dim=1).cpu().numpy()
    rows = np.repeat(np.arange(n), np.diff(g.row_ptr))
    el = g.elabel if g.elabel is not None else np.zeros(m, dtype=np.int32)
    exp = np.unique(np.stack([a[rows], el, b[g.col]], axis=1), axis=0)
    assert np.array_equal(got, exp)
    r.close()
