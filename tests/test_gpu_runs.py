"""GPU tests of the distinct keys of the summary graph's sorted entries: runs
that end at, before and after a wave's rows and a tile, one run, no repeats.

Reference: numpy's unique rows.
"""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m", [1, 63, 64, 65, 1023, 1024, 1025, 4095, 4096, 4097, 3 * 4096 + 1])
@pytest.mark.parametrize("run", [1, 3, 64, 4096, 1 << 20])
def test_runs(m, run):
    import paper_2204_05821_amd as kb
    n = 97
    rng = np.random.default_rng(m * 7 + run)
    src = np.sort(rng.integers(0, n, m))
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(src, minlength=n), out=rp[1:])
    lab = (np.arange(m) // run).astype(np.int32)  # one block on both sides: `run` entries per key
    t = lambda x, d: torch.from_numpy(np.ascontiguousarray(x, dtype=d)).cuda()
    r = kb.Refiner(t(rp, np.int64), t(np.zeros(m), np.int32), t(lab, np.int32), kmax=1)
    zero = t(np.zeros(n), np.int32)
    got = np.stack([x.cpu().numpy() for x in r.quotient(zero, zero)], axis=1)
    r.close()
    exp = np.unique(np.stack([np.zeros(m, np.int32), lab, np.zeros(m, np.int32)], axis=1), axis=0)
    assert np.array_equal(got, exp)
