"""The device-built degree schedule at the edges of its chunks (16,384 vertices), ranges and tiers:
tier totals against the degrees, partitions against the CPU reference."""
from __future__ import annotations

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CHUNK = 16_384


def _tiers(deg, cap, row_max):
    lo, mid, hi = deg <= cap, (deg > cap) & (deg <= row_max), deg > row_max
    return [(int(x.sum()), int(deg[x].sum())) for x in (lo, mid, hi)]


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, CHUNK - 1, CHUNK, CHUNK + 1, 2 * CHUNK + 77])
@pytest.mark.parametrize("key_bits", [0, 64])
@pytest.mark.parametrize("form", ["sparse", "dense", "long", "long_wide_labels"])
def test_tiers_and_partitions(n, key_bits, form):
    import paper_2204_05821_amd as kb
    print(f"[schedule] n={n} keys={key_bits} {form}", flush=True)
    cap, row_max = (2048, 19_456) if key_bits == 0 else (1024, 8192)
    rng = np.random.default_rng(n)
    deg = rng.integers(0, 3, n) if form != "dense" else rng.integers(0, 40, n)
    if form == "sparse":
        deg[: n // 2] = 0
    if form.startswith("long"):
        special = [cap, cap + 1, 4096, 4097, 8192, 8193, row_max, row_max + 1, cap, 1]
        at = [0, 1, 255, 256, n - 1, n - 2, CHUNK - 1, CHUNK, CHUNK - 2, CHUNK + 1]
        for v, d in zip(at, special):
            if 0 <= v < n:
                deg[v] = d
    src = np.repeat(np.arange(n), deg)
    dst = rng.integers(0, n, len(src))
    lab = rng.integers(0, 3, len(src))
    if form == "long_wide_labels":  # labels in an array of their own, moved with the ordered entries
        lab = np.array([0, 12_345, 2**31 - 1])[lab]
    sets = rng.integers(0, 3, n)
    vp = np.concatenate([[0], np.cumsum(sets)])
    g = graphgen.from_edges(n, src, dst, lab, rng.integers(0, 4, int(vp[-1])), vp)
    r = kb.Refiner(*kb.to_device(g), kmax=2, tuning=kb.tuning(key_bits=key_bits))
    info = r.schedule_info()
    lo, mid, hi = _tiers(np.diff(g.row_ptr), cap, row_max)
    assert (info["range"]["vertices"], info["range"]["entries"]) == lo
    assert (info["workgroup"]["vertices"], info["workgroup"]["entries"]) == mid
    assert tuple(info["hub"][k] + info["hub_global"][k] for k in ("vertices", "entries")) == hi
    p0, c0 = r.initial()
    ids, counts = r.refine(2)
    e0, ec0 = oracle.initial(g)
    exp, ec = oracle.refine(g, 2)
    assert c0 == ec0 and counts == ec
    for a, b in zip([p0] + ids, [e0] + exp):
        assert np.array_equal(a.cpu().numpy(), b)
    r.close()
