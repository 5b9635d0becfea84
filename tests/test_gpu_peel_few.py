"""GPU tests of the one-workgroup peeling round around the collisions it takes: fewer, about as
many and more than 4,096 collided vertices, forced by key hashes cut to 8 bits.

Reference: the CPU oracle.
"""
from __future__ import annotations

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [300, 700, 4_300, 4_400, 6_000])
@pytest.mark.parametrize("key_bits", [0, 32])
def test_collisions(n, key_bits, monkeypatch):
    import paper_2204_05821_amd as kb
    print(f"[peel] n={n} keys={key_bits}", flush=True)
    monkeypatch.setenv("KBISIM_DEBUG_HASH_BITS", "8")
    rng = np.random.default_rng(n)
    # one or two entries a vertex with many labels: nearly every signature is its own block
    src = np.concatenate([np.arange(n), rng.integers(0, n, n // 2)])
    g = graphgen.from_edges(n, src, rng.integers(0, n, len(src)), rng.integers(0, n, len(src)),
                            rng.integers(0, 4, n), np.arange(n + 1))
    r = kb.Refiner(*kb.to_device(g), kmax=2, tuning=kb.tuning(key_bits=key_bits))
    ids, counts = r.refine(2)
    exp, ec = oracle.refine(g, 2)
    assert counts == ec
    for a, b in zip(ids, exp):
        assert np.array_equal(a.cpu().numpy(), b)
    r.close()
