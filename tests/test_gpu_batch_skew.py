"""Batches of graphs of very different sizes (GPU): graph ids and the check that entries stay inside
their graph, at the edges of the chunks of 4,096 vertices and entries, and the time that one large
graph takes among thousands of small ones."""
from __future__ import annotations

import time

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _union(sizes, seed):
    """Graphs of the given (vertices, entries), their union's arrays and vertex offsets."""
    import paper_2204_05821_amd as kb
    gs = []
    for i, (n, m) in enumerate(sizes):
        src, dst = graphgen.uniform_edges(n, m, seed + i) if m else (np.zeros(0, np.int32), np.zeros(0, np.int32))
        gs.append(graphgen.from_edges(n, src, dst, None, None))
    return gs, kb.union_of(gs)


SIZES = {
    "whole_chunks": [(4096, 4096), (4096, 8192), (1, 0), (4095, 4097)],
    "many_in_a_chunk": [(0, 0)] * 5_000 + [(1, 1), (0, 0), (2, 0), (1, 3)] * 2_000 + [(0, 0)] * 5_000,
    "large_among_small": [(2, 2)] * 3_000 + [(0, 0), (30_011, 100_003)] + [(3, 1)] * 3_000,
    "one": [(1, 2)],
}


@pytest.mark.parametrize("name", SIZES)
def test_ids_and_bounds(name):
    import paper_2204_05821_amd as kb
    print(f"[batch skew] {name}", flush=True)
    gs, (rp, col, el, vl, vp, off) = _union(SIZES[name], 3)
    dev = lambda a: None if a is None else torch.from_numpy(a).cuda()
    b = kb.Batch(dev(rp), dev(col), dev(el), dev(vl), dev(vp), off, kmax=2)
    ids, counts = b.refine(2)
    b.close()
    ids = [x.cpu().numpy() for x in ids]
    for g in range(0, len(gs), max(1, len(gs) // 200)):
        exp, ec = oracle.refine(gs[g], 2)
        assert list(counts[g]) == ec
        for a, e in zip(ids, exp):
            assert np.array_equal(a[off[g]:off[g + 1]], e)
    # one entry that leaves its graph, where chunks and graphs begin and end
    m = len(col)
    graph = np.searchsorted(np.asarray(off), np.repeat(np.arange(len(rp) - 1), np.diff(rp)), side="right") - 1
    for e in sorted({0, m // 2, m - 1, *(x for x in (4095, 4096, 8191, 8192) if x < m)}):
        for bad in (off[graph[e]] - 1, off[graph[e] + 1]):
            if not 0 <= bad < off[-1]:
                continue
            c2 = col.copy()
            c2[e] = bad
            with pytest.raises(kb.KbisimError) as ei:
                kb.Batch(dev(rp), dev(c2), dev(el), dev(vl), dev(vp), off, kmax=2)
            assert ei.value.code == kb.EGRAPH
    # row offsets out of order are refused, not followed
    if len(rp) > 3:
        r2 = rp.copy()
        r2[1], r2[-2] = m, 0
        with pytest.raises(kb.KbisimError) as ei:
            kb.Batch(dev(r2), dev(col), dev(el), dev(vl), dev(vp), off, kmax=2)
        assert ei.value.code == kb.EGRAPH


def test_large_graph_among_small_ones():
    """Creating the batch takes about as long as with the small graphs counted as one."""
    import paper_2204_05821_amd as kb
    small, n, m = 9_000, 4_000_000, 40_000_000
    gen = torch.Generator(device="cuda").manual_seed(1)
    tail = torch.arange(small, device="cuda")
    deg = torch.bincount(torch.randint(0, n, (m,), generator=gen, device="cuda"), minlength=n)
    deg = torch.cat([deg, torch.ones(2 * small, device="cuda", dtype=deg.dtype)])
    rp = torch.zeros(n + 2 * small + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(deg, 0, out=rp[1:])
    col = torch.cat([torch.randint(0, n, (m,), generator=gen, device="cuda", dtype=torch.int32),
                     (n + 2 * tail).repeat_interleave(2).int()])
    del deg

    def create(off):
        best = 1e9
        for _ in range(3):
            torch.cuda.synchronize()
            t = time.perf_counter()
            b = kb.Batch(rp, col, None, None, None, off, kmax=1)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
            b.close()
        return best

    few = create([0, n, n + 2 * small])
    many = create([0] + [n + 2 * i for i in range(small + 1)])
    print(f"[batch skew] create: 2 graphs {few * 1e3:.2f} ms, {small + 1} graphs {many * 1e3:.2f} ms", flush=True)
    assert many < 3 * few
