"""Calls of many steps (GPU): epochs laid out in segments of 14 steps, wraps across calls, tile counts
scanned by the assign kernel (up to 256 tiles) or by a launch of their own."""
from __future__ import annotations

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _check(r, g, k, start=None):
    exp, ec = oracle.refine(g, k)
    ids, counts = r.refine(k)
    assert counts == ec, k
    for a, b in zip(ids, exp):
        assert np.array_equal(a.cpu().numpy(), b)


@pytest.mark.parametrize("graphs", [False, True])
def test_segments_and_wraps(graphs):
    import paper_2204_05821_amd as kb
    g = graphgen.deep(seed=12, n=3_000, avg_degree=1.05)
    r = kb.Refiner(*kb.to_device(g), kmax=33, graphs=graphs)
    for k in (1, 13, 14, 15, 14, 1, 28, 29, 33, 2, 14):
        print(f"[steps] graphs={graphs} k={k}", flush=True)
        _check(r, g, k)
    r.close()


def test_collisions_in_a_later_segment(monkeypatch):
    """Truncated hashes: steps of every segment are redone with host-driven rounds."""
    import paper_2204_05821_amd as kb
    for bits in (4, 12):
        monkeypatch.setenv("KBISIM_DEBUG_HASH_BITS", str(bits))
        g = graphgen.deep(seed=13, n=1_500, avg_degree=1.1)
        r = kb.Refiner(*kb.to_device(g), kmax=20)
        for k in (20, 15, 3):
            _check(r, g, k)
        r.close()


@pytest.mark.parametrize("items", [8, 16])
@pytest.mark.parametrize("tiles", [1, 255, 256, 257])
@pytest.mark.parametrize("extra", [0, 1])
def test_tile_counts(items, tiles, extra):
    import paper_2204_05821_amd as kb
    n = tiles * 256 * items + extra
    print(f"[steps] tiles={tiles} items={items} n={n}", flush=True)
    rng = np.random.default_rng(n)
    vl = rng.integers(0, n, n).astype(np.int32)
    rp = np.zeros(n + 1, dtype=np.int64)
    r = kb.Refiner(torch.from_numpy(rp).cuda(), torch.zeros(0, dtype=torch.int32, device="cuda"), None,
                   torch.from_numpy(vl).cuda(), kmax=1, tuning=kb.tuning(scan_items=items))
    ids, counts = r.refine(1)
    _, first, inv = np.unique(vl, return_index=True, return_inverse=True)
    new = np.empty(len(first), dtype=np.int64)
    new[np.argsort(first)] = np.arange(len(first))
    assert counts == [len(first)]
    assert np.array_equal(ids[0].cpu().numpy(), new[inv])
    r.close()
