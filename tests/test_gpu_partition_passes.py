"""Grouping by partition (GPU) where a bucket holds more keys than one workgroup's set, against the
CPU reference: few bucket bits on a small graph put up to 30,000 distinct keys in a bucket (the set
is marked full at 3,072 of 4,096 slots), so whole passes overflow and are split again and again, or
begin split where that is planned for (the second number: bucket bits of the plan)."""
from __future__ import annotations

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def twins(half, seed):
    """Rows of two or three labelled entries, nearly all different; row half + i repeats row i."""
    rng = np.random.default_rng(seed)
    deg = rng.integers(2, 4, half)
    src = np.repeat(np.arange(half), deg)
    dst, lab = rng.integers(0, 2 * half, len(src)), rng.integers(0, 1 << 20, len(src))
    return graphgen.from_edges(2 * half, np.concatenate([src, src + half]), np.concatenate([dst, dst]),
                               np.concatenate([lab, lab]), None, name=f"twins_{half}")


@pytest.mark.parametrize("bits", ["0", "2", "3", "6", "0,0", "2,2", "3,1", "2,4", "6,6"])
@pytest.mark.parametrize("half", [6_000, 30_000])
def test_overflowing_buckets(half, bits, monkeypatch):
    import paper_2204_05821_amd as kb
    print(f"[partition passes] half={half} bits={bits}", flush=True)
    monkeypatch.setenv("KBISIM_DEBUG_GROUP_MIN", "1")
    monkeypatch.setenv("KBISIM_DEBUG_GROUP_BITS", bits)
    g = twins(half, len(bits))
    exp, ec = oracle.refine(g, 3)
    assert ec[0] > 0.99 * half
    r = kb.refiner_for(g, kmax=3)
    ids, counts = r.refine(3)
    assert counts == ec
    for a, b in zip(ids, exp):
        assert np.array_equal(a.cpu().numpy(), b)
    r.close()


@pytest.mark.parametrize("n", [4_097, 10_240, 10_241, 30_011])  # rows, in ranges of 256
@pytest.mark.parametrize("shared", [1.0, 0.5])
@pytest.mark.parametrize("hash_bits", [None, 12])
def test_key_shared_by_a_tile(n, shared, hash_bits, monkeypatch):
    """One key for many rows: one per range reaches the second pass, and where that makes over 40 in a
    tile of 4,096 pairs all but one of them drop out.  With 12 hash bits other keys collide with it."""
    import paper_2204_05821_amd as kb
    print(f"[shared key] n={n} shared={shared} bits={hash_bits}", flush=True)
    monkeypatch.setenv("KBISIM_DEBUG_GROUP_MIN", "1")
    if hash_bits is not None:
        monkeypatch.setenv("KBISIM_DEBUG_HASH_BITS", str(hash_bits))
    rng = np.random.default_rng(n)
    lab = np.where(rng.random(n) < shared, 0, rng.integers(1, 1 << 20, n))
    g = graphgen.from_edges(n, np.arange(n), rng.integers(0, n, n), lab, None, name=f"shared_{n}_{shared}")
    exp, ec = oracle.refine(g, 3)
    r = kb.refiner_for(g, kmax=3)
    ids, counts = r.refine(3)
    assert counts == ec
    for a, b in zip(ids, exp):
        assert np.array_equal(a.cpu().numpy(), b)
    r.close()


@pytest.mark.parametrize("n", [9_000, 40_000])
def test_table_calls_between_partitioned_ones(n, monkeypatch):
    """The table, cleared only where partitioned steps wrote, over many epochs: work-efficient calls and
    updates among refine calls of odd lengths, each against the reference."""
    import paper_2204_05821_amd as kb
    from tests.test_gpu_incremental import edited
    print(f"[table between] n={n}", flush=True)
    monkeypatch.setenv("KBISIM_DEBUG_GROUP_MIN", "1")
    rng = np.random.default_rng(n)
    src, dst = graphgen.uniform_edges(n, n + n // 4, 5)
    g = graphgen.from_edges(n, src, dst, None, rng.integers(0, 3, n), name=f"sparse_{n}")
    chain = [oracle.refine(g, k) for k in range(1, 10)]
    r = kb.refiner_for(g, kmax=9)
    for turn in range(12):
        for k, mode in ((1 + turn % 9, True), (9 - turn % 5, False), (3 + turn % 4, False), (1 + turn % 3, True)):
            r.work_efficient(mode)
            ids, counts = r.refine(k)
            exp, ec = chain[k - 1]
            assert counts == ec, (turn, k, mode)
            for a, b in zip(ids, exp):
                assert np.array_equal(a.cpu().numpy(), b)
    r.work_efficient(False)
    r.incremental()
    for turn in range(6):
        ids, counts = r.refine(9)
        assert counts == chain[8][1]
        g2, rows = edited(g, rng, 5, 5)
        e2, c2 = oracle.refine(g2, 9)
        rp, col, el, _, _ = kb.to_device(g2)
        ids, counts = r.update(rp, col, el, torch.from_numpy(rows).cuda(), 9)
        assert counts == c2
        for a, b in zip(ids, e2):
            assert np.array_equal(a.cpu().numpy(), b)
    r.close()
