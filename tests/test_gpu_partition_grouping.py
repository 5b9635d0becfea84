"""Grouping by partition (GPU) against the CPU reference, forced on small graphs: keys of single
vertices, keys shared by most vertices (dropped per tile), truncated hashes (collisions, one bucket),
label sets, hubs, batches, graph replay, updates and work-efficient calls on the same context."""
from __future__ import annotations

import numpy as np
import pytest

import graphgen
import oracle
from tests.test_gpu_incremental import edited
from tests.test_gpu_parity import tier_graph

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _graphs():
    yield graphgen.tiny(seed=5, n=4_100, m=9_000)
    yield graphgen.rmat(14, 300_000, seed=6)
    yield graphgen.rmat_rdf(13, 90_000, seed=7, types=100, elabels=1000)
    yield graphgen.deep(seed=8, n=30_000, avg_degree=1.6)
    src, dst = graphgen.uniform_edges(70_001, 400_000, 9)  # one key at first, then few
    yield graphgen.from_edges(70_001, src, dst, None, None, name="one_key")
    yield tier_graph(seed=10, labels=20, shared_targets=500)


def _same(ids, counts, exp, ec):
    assert counts == ec
    for a, b in zip(ids, exp):
        assert np.array_equal(a.cpu().numpy(), b)


@pytest.mark.parametrize("bits", [None, 0, 3, 14, 20])
@pytest.mark.parametrize("replay", [False, True])
def test_refine(bits, replay, monkeypatch):
    import paper_2204_05821_amd as kb
    monkeypatch.setenv("KBISIM_DEBUG_GROUP_MIN", "1")
    if bits is not None:
        monkeypatch.setenv("KBISIM_DEBUG_HASH_BITS", str(bits))
    for g in _graphs():
        if bits is not None and bits < 14 and g.m > 100_000:
            continue
        print(f"[partition] {g.name} bits={bits} replay={replay}", flush=True)
        exp, ec = oracle.refine(g, 4)
        r = kb.Refiner(*kb.to_device(g), kmax=4, graphs=replay)
        for _ in range(2):
            _same(*r.refine(4), exp, ec)
        r.close()


def test_table_users_after_partitioned_steps(monkeypatch):
    import paper_2204_05821_amd as kb
    monkeypatch.setenv("KBISIM_DEBUG_GROUP_MIN", "1")
    rng = np.random.default_rng(3)
    for g in _graphs():
        print(f"[partition] {g.name}", flush=True)
        exp, ec = oracle.refine(g, 4)
        r = kb.Refiner(*kb.to_device(g), kmax=4)
        _same(*r.refine(4), exp, ec)
        r.work_efficient(True)
        _same(*r.refine(4), exp, ec)
        r.work_efficient(False)
        r.incremental()
        _same(*r.refine(4), exp, ec)
        g2, rows = edited(g, rng, 5, 5)
        e2, c2 = oracle.refine(g2, 4)
        for _ in range(2):
            rp, col, el, _, _ = kb.to_device(g2)
            _same(*r.update(rp, col, el, torch.from_numpy(rows).cuda(), 4), e2, c2)
            _same(*r.refine(4), exp, ec)
        r.close()


def test_batch(monkeypatch):
    import paper_2204_05821_amd as kb
    monkeypatch.setenv("KBISIM_DEBUG_GROUP_MIN", "1")
    gs = [graphgen.batch_graph(i, m) for i, m in enumerate([1_000, 30_000, 5_000, 80_000])]
    b = kb.batch_for(gs, kmax=3)
    ids, counts = b.refine(3)
    at = 0
    for g, cnt in zip(gs, counts):
        _same([x[at:at + g.n] for x in ids], cnt, *oracle.refine(g, 3))
        at += g.n
    b.close()
