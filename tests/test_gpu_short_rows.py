"""Exact check of short rows (GPU) against the CPU reference: rows around the groups of four and eight
entries that are read together, each beside a permutation of itself, a row that lacks one of its pairs
(another one twice instead) and a row with one pair changed; key hashes cut to 0 bits leave every
decision to the check, through the table's lookups, the partition and the peeling round.  And vertices
without entries around the 4,096 that one workgroup takes."""
from __future__ import annotations

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _check(g, k):
    import paper_2204_05821_amd as kb
    exp, ec = oracle.refine(g, k)
    r = kb.refiner_for(g, kmax=k)
    ids, counts = r.refine(k)
    assert counts == ec
    for a, b in zip(ids, exp):
        assert np.array_equal(a.cpu().numpy(), b)
    r.close()


@pytest.mark.parametrize("lengths", [(1, 2), (3, 4, 5), (7, 8, 9), (12, 13, 15, 16)])
@pytest.mark.parametrize("partition", [False, True])
@pytest.mark.parametrize("bits", [0, None])
def test_near_equal_rows(lengths, partition, bits, monkeypatch):
    print(f"[short rows] lengths={lengths} partition={partition} bits={bits}", flush=True)
    if partition:
        monkeypatch.setenv("KBISIM_DEBUG_GROUP_MIN", "1")
    if bits is not None:
        monkeypatch.setenv("KBISIM_DEBUG_HASH_BITS", str(bits))
    rng = np.random.default_rng(lengths[0])
    rows = []
    for _ in range(40):
        for length in lengths:
            row = list(zip(rng.permutation(1_000)[:length], rng.integers(0, 3, length)))
            rows.append(row)
            rows.append([row[i] for i in rng.permutation(length)])
            if length > 1:
                rows.append(row[:-1] + [row[0]])
                rows.append(row + [row[0]])
            rows.append(row[:-1] + [(row[-1][0], 7)])
    order = rng.permutation(len(rows))
    src = np.repeat(np.arange(len(rows)), [len(rows[i]) for i in order])
    dst, lab = np.array([e for i in order for e in rows[i]]).T
    n = 1_000 + len(rows)
    g = graphgen.from_edges(n, src + 1_000, dst, lab, np.concatenate([np.arange(1_000) % 50, np.full(len(rows), 60)]))
    _check(g, 2)


@pytest.mark.parametrize("n", [1, 4_095, 4_096, 4_097, 20_483])
@pytest.mark.parametrize("labels", [1, 3, 10_000])
@pytest.mark.parametrize("partition", [False, True])
def test_rows_without_entries(n, labels, partition, monkeypatch):
    print(f"[empty rows] n={n} labels={labels} partition={partition}", flush=True)
    if partition:
        monkeypatch.setenv("KBISIM_DEBUG_GROUP_MIN", "1")
    rng = np.random.default_rng(n)
    m = n // 3
    _check(graphgen.from_edges(n, rng.integers(0, n, m), rng.integers(0, n, m), None, rng.integers(0, labels, n)), 3)
