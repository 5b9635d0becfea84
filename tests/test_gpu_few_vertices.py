"""Graphs of few vertices and many entries (GPU): in-degree ranking on both sides of its line, and the
time of creating one against a graph of as many entries and more vertices."""
from __future__ import annotations

import time

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [2, 4, 5, 9, 130])
@pytest.mark.parametrize("skew", [False, True])
def test_few_vertices(n, skew):
    import paper_2204_05821_amd as kb
    m = (1 << 21) + 77
    print(f"[few vertices] n={n} skew={skew}", flush=True)
    rng = np.random.default_rng(n)
    src, dst, lab = rng.integers(0, n, m), rng.integers(0, n, m), rng.integers(0, 3, m)
    if skew:  # one target of nearly all entries, two rows of few
        dst[1_000:] = n - 1
        src[m // 2:] = 0
    lab[src == 1] = 0
    g = graphgen.from_edges(n, src, dst, lab)
    exp, ec = oracle.refine(g, 3)
    r = kb.refiner_for(g, kmax=3)
    ids, counts = r.refine(3)
    assert counts == ec
    for a, b in zip(ids, exp):
        assert np.array_equal(a.cpu().numpy(), b)
    r.close()


def test_create_time():
    import paper_2204_05821_amd as kb
    m = 30_000_000

    def create(n):
        col = torch.randint(0, n, (m,), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda",
                            dtype=torch.int32)
        rp = (torch.arange(n + 1, device="cuda") * m) // n
        best = 1e9
        for _ in range(3):
            torch.cuda.synchronize()
            t = time.perf_counter()
            r = kb.Refiner(rp, col, kmax=1)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
            r.close()
        return best

    few, many = create(2), create(100_000)
    print(f"[few vertices] create: 2 vertices {few * 1e3:.2f} ms, 100,000 vertices {many * 1e3:.2f} ms", flush=True)
    assert few < 3 * many
