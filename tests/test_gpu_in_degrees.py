"""In-degree ranking of large graphs (targets partitioned into buckets) at the edges of its paths.

An unlabelled graph's first partitions have a closed form: P_1 separates the
vertices with entries, P_2 further by which of the two blocks their targets
are in, and P_3 by which of those.  A target counted as unnamed would be
missing from the gathers, so the partitions would differ.
"""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

M = 1 << 21  # entries from which targets are partitioned


def _canonical(key):
    _, first, inv = np.unique(key, return_index=True, return_inverse=True)
    order = np.argsort(first)
    new = np.empty_like(order)
    new[order] = np.arange(len(order))
    return new[inv].astype(np.int32)


# counters of 2^13 and 2^15 targets per bucket, one pass and two; hub: a bucket past its share
@pytest.mark.parametrize("n", [1, 300, 1 << 21, (1 << 21) + 1, 1 << 23, (1 << 23) + 5])
@pytest.mark.parametrize("m", [M - 1, M, M + 8191])
@pytest.mark.parametrize("hub", [False, True])
def test_first_partitions(n, m, hub):
    import paper_2204_05821_amd as kb
    print(f"[in-degrees] n={n} m={m} hub={hub}", flush=True)
    rng = np.random.default_rng(n + m)
    src = np.sort(rng.integers(0, max(1, n - n // 3), m))
    dst = rng.integers(n // 5, n, m).astype(np.int32)
    if hub:
        dst[m // 4:] = n - 1
        dst[: m // 8] = n // 5
    rp = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(src, minlength=n), out=rp[1:])
    r = kb.Refiner(torch.from_numpy(rp).cuda(), torch.from_numpy(dst).cuda(), kmax=3)
    ids, _ = r.refine(3)
    pid = np.zeros(n, dtype=np.int64)
    for got in ids:
        assert pid.max() < 32  # one bit per block in the reference's key
        key = pid << 32
        for b in range(int(pid.max()) + 1):
            has = np.zeros(n, dtype=bool)
            has[src[pid[dst] == b]] = True
            key = key + (has.astype(np.int64) << b)
        pid = _canonical(key).astype(np.int64)
        assert np.array_equal(got.cpu().numpy(), pid)
    r.close()
