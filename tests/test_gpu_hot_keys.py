"""Vertices that share few keys (GPU) against the CPU reference, bit-exact.

The grouping tables take one insert per key of a wave: from one label for all
vertices to more labels than a wave's meeting slots, unlabelled sparse graphs,
ragged sizes, and an update whose edits touch the large blocks of vertices
without entries.
"""
from __future__ import annotations

import numpy as np
import pytest

import graphgen
import oracle
from tests.test_gpu_incremental import edited

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _graph(n, m, labels, seed=3):
    src, dst = graphgen.uniform_edges(n, m, seed)
    vl = graphgen.vertex_labels(n, labels, 0.0, seed) if labels else None
    return graphgen.from_edges(n, src, dst, None, vl, name=f"hot_n{n}_l{labels}")


@pytest.mark.parametrize("n,m,labels", [(1, 0, 1), (63, 20, 0), (65, 65, 2), (257, 300, 3), (20_011, 9_000, 1),
                                        (20_011, 24_000, 0), (20_011, 24_000, 255), (20_011, 24_000, 5_000)])
def test_few_keys(n, m, labels):
    import paper_2204_05821_amd as kb
    g = _graph(n, m, labels)
    print(f"[hot keys] {g.name} m={m}", flush=True)
    r = kb.refiner_for(g, kmax=6)
    p0, c0 = r.initial()
    ids, counts = r.refine(6)
    e0, ec0 = oracle.initial(g)
    exp, ec = oracle.refine(g, 6)
    assert c0 == ec0 and counts == ec
    assert np.array_equal(p0.cpu().numpy(), e0)
    for a, b in zip(ids, exp):
        assert np.array_equal(a.cpu().numpy(), b)
    r.close()


@pytest.mark.parametrize("labels", [0, 1, 300])
def test_update_of_large_empty_blocks(labels):
    import paper_2204_05821_amd as kb
    g = _graph(50_021, 20_000, labels)
    empty = np.flatnonzero(np.diff(g.row_ptr) == 0)
    g2, rows = edited(g, np.random.default_rng(5), 4, 3, fill_rows=[int(empty[7]), int(empty[-1])])
    r = kb.refiner_for(g, kmax=5)
    r.incremental()
    r.refine(5)
    rp, col, el, _, _ = kb.to_device(g2)
    ids, counts = r.update(rp, col, el, torch.from_numpy(rows).cuda(), 5)
    exp, ec = oracle.refine(g2, 5)
    assert counts == ec
    for a, b in zip(ids, exp):
        assert np.array_equal(a.cpu().numpy(), b)
    r.close()
