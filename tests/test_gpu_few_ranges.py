"""GPU tests of the range kernel's two widths at the number of ranges where
one takes over from the other: single-row ranges, ranges of full vertex count
and of full entry count, with exact and hashed 32-bit keys.

Reference: the CPU oracle.
"""
from __future__ import annotations

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FEW = 512


@pytest.mark.parametrize("ranges", [1, FEW, FEW + 1])
@pytest.mark.parametrize("form", ["rows", "vertices", "entries"])
@pytest.mark.parametrize("key_bits", [0, 32])
def test_widths(ranges, form, key_bits):
    import paper_2204_05821_amd as kb
    print(f"[few ranges] {ranges} {form} {key_bits}", flush=True)
    rng = np.random.default_rng(ranges)
    rows, d = {"rows": (1, 2048), "vertices": (256, 1), "entries": (128, 16)}[form]
    n = ranges * rows
    src = np.repeat(np.arange(n), d)
    g = graphgen.from_edges(n, src, rng.integers(0, n, n * d), rng.integers(0, 3, n * d), rng.integers(0, 4, n),
                            np.arange(n + 1))
    r = kb.Refiner(*kb.to_device(g), kmax=2, tuning=kb.tuning(key_bits=key_bits))
    ids, counts = r.refine(2)
    exp, ec = oracle.refine(g, 2)
    assert counts == ec
    for a, b in zip(ids, exp):
        assert np.array_equal(a.cpu().numpy(), b)
    r.close()
