"""GPU tests of the one-workgroup peeling round over rows of every kind: empty, compared by a thread
(up to 16 entries), by the workgroup (longer), twins among them; key hashes cut to few bits make all
of them collide.  Reference: the CPU oracle."""
from __future__ import annotations

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("lengths", [(1,), (16, 17), (0, 1, 16, 17, 40), (3, 300, 1_100)])
@pytest.mark.parametrize("n", [130, 1_500])
@pytest.mark.parametrize("bits", [0, 5, 12])
def test_collided_rows(lengths, n, bits, monkeypatch):
    import paper_2204_05821_amd as kb
    print(f"[peel rows] n={n} lengths={lengths} bits={bits}", flush=True)
    monkeypatch.setenv("KBISIM_DEBUG_HASH_BITS", str(bits))
    rng = np.random.default_rng(n + bits)
    deg = rng.choice(lengths, n)
    src = np.repeat(np.arange(n), deg)
    dst, lab = rng.integers(0, 2 * n, len(src)), rng.integers(0, 3, len(src))
    g = graphgen.from_edges(2 * n, np.concatenate([src, src + n]), np.concatenate([dst, dst]),
                            np.concatenate([lab, lab]), np.tile(rng.integers(0, 2, n), 2), None)
    r = kb.refiner_for(g, kmax=3)
    ids, counts = r.refine(3)
    exp, ec = oracle.refine(g, 3)
    assert counts == ec
    for a, b in zip(ids, exp):
        assert np.array_equal(a.cpu().numpy(), b)
    r.close()
