"""The cases this library's speed is measured on, through its public Python entry points.

Each case is one thing a user of the library has it do on one GPU: refine a
graph kept on the device, refine a new graph once (context creation
included), refine many graphs as one batch, refine the inverse graph, build
the summary graph, update a cached chain after edits.  Sizes and label
distributions are those of the benchmark and the test recipes (uniform,
RMAT, RDF-like RMAT, batches of mixed graphs), with seeded random inputs made
on the GPU.  All outputs are whole numbers (block ids and counts).
"""
from __future__ import annotations

import math

import torch

import paper_2204_05821_amd as kb
from paper_2204_05821_amd import presets

DEV = "cuda"
CHUNK = 1 << 26  # entries generated at a time


# ---------------------------------------------------------------- cases
def listed():
    return [
        # the smallest graphs: launches and latency are all there is.  A one-off
        # summary of a small graph (the context is created and dropped) ...
        dict(name="oneshot_uniform_10k", op="oneshot", kind="uniform", n=10_000, m=50_000, vlabels=4, elabels=8, k=10),
        # ... and repeated refinements on a kept context
        dict(name="refine_uniform_10k", op="refine", kind="uniform", n=10_000, m=50_000, vlabels=4, elabels=8, k=10),
        # a sparse unlabelled graph that keeps refining through every step, odd sizes
        dict(name="refine_sparse_1M", op="refine", kind="uniform", n=1_000_003, m=1_200_007, vlabels=0, elabels=0, k=10),
        # an ordinary graph of a serving pool: created, refined and returned once
        dict(name="oneshot_rmat_24M", op="oneshot", kind="rmat", n=1 << 21, m=23_456_789, vlabels=32, elabels=64, k=5),
        # the 100M-edge graph (the size of the smaller published datasets)
        dict(name="refine_rmat_100M", op="refine", kind="rmat", n=1 << 23, m=100_000_000, vlabels=32, elabels=64, k=10),
        # the largest: the RDF-like graph of 10^9 edges with type-label sets
        dict(name="refine_rdf_1B", op="refine", kind="rdf", n=1 << 27, m=1_000_000_000, vlabels=1000, elabels=1000, k=10),
        # a cohort of small served jobs: one batch created, refined and returned
        dict(name="batch_oneshot_64", op="batch_oneshot", graphs=64, lo=1_000, hi=200_000, vlabels=16, elabels=32, k=10),
        # a large batch kept on the device, its step loop replayed as a HIP graph
        dict(name="batch_refine_1024", op="batch_refine", graphs=1024, lo=1_000, hi=2_000_000, vlabels=16, elabels=32,
             k=10),
        # backward bisimulation with all labels: transpose, create, refine
        dict(name="backward_rmat_40M", op="backward", kind="rmat", n=1 << 22, m=40_000_003, vlabels=32, elabels=64, k=5),
        # the summary graph of P_k over P_{k-1}
        dict(name="quotient_rdf_125M", op="quotient", kind="rdf", n=1 << 24, m=125_000_000, vlabels=1000, elabels=1000,
             k=5),
        # an evolving graph: the partitions after 1,000 edited entries
        dict(name="update_rmat_100M", op="update", kind="rmat", n=1 << 23, m=100_000_000, vlabels=32, elabels=64, k=10,
             edits=1000),
        # all partitions with singleton blocks skipped and a stop at the fixpoint
        dict(name="work_efficient_rdf_250M", op="work_efficient", kind="rdf", n=1 << 25, m=250_000_000, vlabels=1000,
             elabels=1000, k=10),
    ]


def draw(rng):
    """One more case of the same ranges: log-uniform sizes, power-of-two (RMAT) and odd (uniform) vertex counts."""
    def logu(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["oneshot", "refine", "refine", "batch_oneshot", "batch_refine", "backward", "quotient", "update",
                     "work_efficient"])
    k = rng.randint(1, 10)
    if op in ("batch_oneshot", "batch_refine"):
        hi = logu(20_000, 200_000 if op == "batch_oneshot" else 2_000_000)
        graphs = logu(8, 96 if op == "batch_oneshot" else 1024)
        return dict(op=op, graphs=graphs, lo=1_000, hi=hi, vlabels=16, elabels=32, k=k)
    top = {"oneshot": 50_000_000, "refine": 1_000_000_000, "backward": 50_000_000, "quotient": 125_000_000,
           "update": 100_000_000, "work_efficient": 250_000_000}[op]
    m = logu(10_000, top)
    kind = rng.choice(["uniform", "rmat", "rdf"])
    n = max(16, int(m / rng.uniform(4.0, 12.0)))
    if kind == "uniform":
        vlabels, elabels = rng.choice([(4, 8), (0, 8), (16, 0), (0, 0), (32, 64)])
    else:
        n = 1 << max(4, n.bit_length() - rng.randint(0, 1))
        vlabels, elabels = (32, 64) if kind == "rmat" else (1000, 1000)
    c = dict(op=op, kind=kind, n=n, m=m, vlabels=vlabels, elabels=elabels, k=max(k, 2) if op == "quotient" else k)
    if op == "update":
        c["edits"] = logu(1, 10_000)
    return c


# ---------------------------------------------------------------- inputs
def _zipf(gen, cnt, labels, s):
    """cnt labels in [0, labels): Zipf(s), or uniform for s = 0."""
    if s == 0.0:
        return torch.randint(0, labels, (cnt,), generator=gen, device=DEV, dtype=torch.int32)
    w = torch.arange(1, labels + 1, device=DEV, dtype=torch.float64) ** -s
    cdf = (torch.cumsum(w, 0) / w.sum()).float()
    out = torch.empty(cnt, dtype=torch.int32, device=DEV)
    for a in range(0, cnt, CHUNK):
        u = torch.rand(min(CHUNK, cnt - a), generator=gen, device=DEV)
        out[a:a + CHUNK] = torch.bucketize(u, cdf, out_int32=True).clamp_(max=labels - 1)
    return out


def _scrambled(x, scale):
    """A fixed bijection of [0, 2^scale) (int64), so that RMAT's hot vertices lie anywhere."""
    mask, h = (1 << scale) - 1, (scale + 1) // 2
    x = (x * 0x2545F491 + 0x1234567) & mask
    x ^= x >> h
    return (x * 0x9E3779B1) & mask


def _rmat_bits(gen, cnt, scale, given=None):
    """RMAT (.57, .19, .19, .05): source ids, or target ids given the source ids."""
    out = torch.zeros(cnt, dtype=torch.int64, device=DEV)
    for level in range(scale):
        u = torch.rand(cnt, generator=gen, device=DEV)
        if given is None:
            bit = u < 0.24
        else:
            bit = u < torch.where(((given >> level) & 1) > 0, 0.05 / 0.24, 0.25)
        out |= bit.long() << level
    return out


def _graph(kind, n, m, gen):
    """(row_ptr, col) of a random graph: sources first (their counts give the rows), then each entry's target."""
    if kind == "uniform":
        src = torch.randint(0, n, (m,), generator=gen, device=DEV, dtype=torch.int64)
        deg = torch.bincount(src, minlength=n)
        col = torch.randint(0, n, (m,), generator=gen, device=DEV, dtype=torch.int32)
    else:
        scale = n.bit_length() - 1
        cnt = torch.zeros(n, dtype=torch.int64, device=DEV)
        for a in range(0, m, CHUNK):
            cnt += torch.bincount(_rmat_bits(gen, min(CHUNK, m - a), scale), minlength=n)
        raw = torch.empty(n, dtype=torch.int64, device=DEV)  # unscrambled id of each vertex
        ids = torch.arange(n, device=DEV, dtype=torch.int64)
        raw[_scrambled(ids, scale)] = ids
        deg = cnt[raw]
        del cnt, ids
        ends = torch.cumsum(deg, 0)
        col = torch.empty(m, dtype=torch.int32, device=DEV)
        for a in range(0, m, CHUNK):
            e = torch.arange(a, min(m, a + CHUNK), device=DEV)
            src = raw[torch.bucketize(e, ends, right=True)]
            col[a:a + CHUNK] = _scrambled(_rmat_bits(gen, e.numel(), scale, given=src), scale).int()
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(deg, 0, out=row_ptr[1:])
    return row_ptr, col


def _labels(case, n, m, gen):
    """(elabel, vlabel, vlabel_ptr): uniform, Zipf, or (rdf) sets of 0-3 types per vertex."""
    kind = case.get("kind", "uniform")
    es, vs = {"uniform": (0.0, 0.0), "rmat": (1.1, 1.0), "rdf": (1.2, 1.0)}[kind]
    el = _zipf(gen, m, case["elabels"], es) if case["elabels"] else None
    if not case["vlabels"]:
        return el, None, None
    if kind != "rdf":
        return el, _zipf(gen, n, case["vlabels"], vs), None
    sizes = torch.bucketize(torch.rand(n, generator=gen, device=DEV), torch.tensor([0.25, 0.80, 0.95], device=DEV))
    ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(sizes, 0, out=ptr[1:])
    return el, _zipf(gen, int(ptr[-1]), case["vlabels"], vs), ptr


def _batch(case, gen):
    """The disjoint union of many graphs, m_g log-uniform; even graphs uniform, odd ones RMAT."""
    G = case["graphs"]  # sizes spread evenly over the logarithm, in a fixed mixed order
    at = [(g * 0.6180339887) % 1.0 for g in range(G)]
    ms = [int(round(case["lo"] * math.exp(u * math.log(case["hi"] / case["lo"])))) for u in at]
    parts, offs, base = [], [0], 0
    for g, m in enumerate(ms):
        if g % 2 == 0:
            n = max(16, m // 8)
            rp, col = _graph("uniform", n, m, gen)
        else:
            n = 1 << max(4, math.ceil(math.log2(m / 8)))
            rp, col = _graph("rmat", n, m, gen)
        parts.append((rp[:-1] + base, col + offs[-1]))
        offs.append(offs[-1] + n)
        base += m
    rp = torch.cat([p[0] for p in parts] + [torch.tensor([base], device=DEV)])
    col = torch.cat([p[1] for p in parts])
    return rp, col, offs


def _edited(rp, col, el, edits, gen):
    """The graph after `edits` edited entries (every other one deleted, the rest added), and the rows they touch."""
    n, m = rp.numel() - 1, col.numel()
    src = torch.repeat_interleave(torch.arange(n, device=DEV, dtype=torch.int32), rp[1:] - rp[:-1])
    pick = torch.randint(0, m, (edits,), generator=gen, device=DEV)
    gone, like = pick[::2], pick[1::2]
    keep = torch.ones(m, dtype=torch.bool, device=DEV)
    keep[gone] = False
    new_src = torch.randint(0, n, (like.numel(),), generator=gen, device=DEV, dtype=torch.int32)
    s2, order = torch.sort(torch.cat([src[keep], new_src]), stable=True)
    col2 = torch.cat([col[keep], col[like]])[order]
    el2 = torch.cat([el[keep], el[like]])[order] if el is not None else None
    rp2 = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(s2, minlength=n), 0, out=rp2[1:])
    return rp2, col2, el2, torch.unique(torch.cat([src[gone], new_src])).int()


def _renumbered(rp, col, el, vl, vp, gen):
    """The same graph under a random permutation of its vertices (block and triple counts stay)."""
    perm = torch.randperm(rp.numel() - 1, generator=gen, device=DEV)  # new id -> old id
    new = torch.empty_like(perm, dtype=torch.int32)
    new[perm] = torch.arange(perm.numel(), device=DEV, dtype=torch.int32)

    def rows(ptr):
        deg = (ptr[1:] - ptr[:-1])[perm]
        out = torch.zeros_like(ptr)
        torch.cumsum(deg, 0, out=out[1:])
        return out, torch.repeat_interleave(ptr[perm] - out[:-1], deg) + torch.arange(int(ptr[-1]), device=DEV)

    rp2, at = rows(rp)
    col, el = new[col[at]], None if el is None else el[at]
    if vp is not None:
        vp, at = rows(vp)
        vl = vl[at]
    elif vl is not None:
        vl = vl[perm]
    return rp2, col, el, vl, vp


def _inputs(case, seed):
    # the summary graph's size depends on the graph: there the seed renumbers one graph's vertices
    fixed = case["op"] == "quotient"
    gen = torch.Generator(device=DEV).manual_seed(17 if fixed else seed)
    if case["op"].startswith("batch"):
        rp, col, offs = _batch(case, gen)
    else:
        rp, col = _graph(case["kind"], case["n"], case["m"], gen)
        offs = None
    el, vl, vp = _labels(case, rp.numel() - 1, col.numel(), gen)
    if fixed:
        rp, col, el, vl, vp = _renumbered(rp, col, el, vl, vp, gen.manual_seed(seed))
    return gen, rp, col, el, vl, vp, offs


def prepare(case, seed):
    """The device graph, and for repeated calls the context (and output arrays) a user's program keeps."""
    op, k = case["op"], case["k"]
    gen, rp, col, el, vl, vp, offs = _inputs(case, seed)
    s = dict(op=op, k=k, graph=(rp, col, el, vl, vp), offs=offs)
    if op in ("refine", "work_efficient", "quotient", "update"):
        s["r"] = r = kb.Refiner(rp, col, el, vl, vp, kmax=k)
        s["out"] = r.alloc_outputs(k)
        if op == "work_efficient":
            r.work_efficient(True)
        elif op == "quotient":
            s["ids"], _ = r.refine(k, out=s["out"])
        elif op == "update":
            r.incremental()
            r.refine(k, out=s["out"])
            s["new"] = _edited(rp, col, el, case["edits"], gen)
    elif op == "batch_refine":
        s["b"] = kb.Batch(rp, col, el, vl, vp, offs, kmax=k, graphs=True)
        s["out"] = s["b"].alloc_outputs(k)
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    op, k = s["op"], s["k"]
    rp, col, el, vl, vp = s["graph"]
    if op in ("refine", "work_efficient"):
        return s["r"].refine(k, out=s["out"])
    if op == "oneshot":
        return kb.refine(rp, col, el, vl, vp, k=k)
    if op == "batch_refine":
        ids, counts = s["b"].refine(k, out=s["out"])
        return ids, torch.tensor(counts)
    if op == "batch_oneshot":
        b = kb.Batch(rp, col, el, vl, vp, s["offs"], kmax=k)
        ids, counts = b.refine(k)
        b.close()
        return ids, torch.tensor(counts)
    if op == "backward":
        r = presets.full(rp, col, el, vl, vp, direction="bw", kmax=k)
        res = r.refine(k)
        r.close()
        return res
    if op == "quotient":
        return s["r"].quotient(s["ids"][k - 1], s["ids"][k - 2])
    new_rp, new_col, new_el, rows = s["new"]
    return s["r"].update(new_rp, new_col, new_el, rows, k, out=s["out"])


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    """Bytes only (there is no arithmetic to speak of).  A step reads every entry's target and label, row offset
    (8), previous block (4) and writes a block id (4) per vertex; steps depend on each other."""
    op, k = case["op"], case["k"]
    if op.startswith("batch"):
        # mean of a log-uniform size; 8 entries per vertex (11 for RMAT's power-of-two counts)
        lo, hi = case["lo"], case["hi"]
        m = case["graphs"] * (hi - lo) / math.log(hi / lo)
        n = m / 7
    else:
        m, n = case["m"], case["n"]
    graph = (8 if case["elabels"] else 4) * m + 8 * n
    steps = k * (graph + 8 * n)
    if op == "backward":
        steps += 2 * graph
    elif op == "quotient":
        steps = graph + 8 * n + 12 * m
    elif op in ("update", "work_efficient"):
        steps = graph + 4 * n * (k + 1)
    return {"bytes": steps, "flops": 0}


# ---------------------------------------------------------------- the same by plain torch
def _dense(cols):
    """Ids of equal rows of several int64 columns, numbered by first row."""
    inv = None
    for c in cols:
        c = torch.unique(c, return_inverse=True)[1]
        inv = c if inv is None else torch.unique(inv * (int(c.max()) + 1) + c, return_inverse=True)[1]
    first = torch.full((int(inv.max()) + 1,), inv.numel(), device=inv.device, dtype=torch.int64)
    first.scatter_reduce_(0, inv, torch.arange(inv.numel(), device=inv.device), "amin")
    order = torch.argsort(first)
    new = torch.empty_like(order)
    new[order] = torch.arange(order.numel(), device=inv.device)
    return new[inv]


def _sets(owner, item, n):
    """Two int64 columns that stand for each owner's set of items (sums of random words over distinct items)."""
    inv = torch.unique(item, return_inverse=True)[1]
    kinds = int(inv.max()) + 1 if inv.numel() else 1
    pairs = torch.unique(owner * kinds + inv)
    gen = torch.Generator(device=DEV).manual_seed(1)
    cols = []
    for _ in range(2):
        word = torch.randint(-(1 << 62), 1 << 62, (kinds,), generator=gen, device=DEV)
        cols.append(torch.zeros(n, dtype=torch.int64, device=DEV).index_add_(0, pairs // kinds, word[pairs % kinds]))
    return cols


def exact(case, seed):
    """Plain refinement of the smaller single-graph cases: 64-bit sums of random words over distinct pairs."""
    if case["op"] not in ("refine", "oneshot", "work_efficient", "backward", "update") or case["m"] > 2_000_000:
        return None
    gen, rp, col, el, vl, vp, _ = _inputs(case, seed)
    if case["op"] == "update":
        rp, col, el, _ = _edited(rp, col, el, case["edits"], gen)
    n = rp.numel() - 1
    src = torch.repeat_interleave(torch.arange(n, device=DEV), rp[1:] - rp[:-1])
    dst, lab = col.long(), torch.zeros_like(src) if el is None else el.long()
    if case["op"] == "backward":
        src, dst = dst, src
    if vl is None:
        pid = torch.zeros(n, dtype=torch.int64, device=DEV)
    else:
        owner = torch.arange(n, device=DEV) if vp is None else torch.repeat_interleave(
            torch.arange(n, device=DEV), vp[1:] - vp[:-1])
        pid = _dense(_sets(owner, vl.long(), n))
    ids, counts = [], []
    for _ in range(case["k"]):
        pid = _dense([pid] + _sets(src, lab * n + pid[dst], n))
        ids.append(pid.int())
        counts.append(int(pid.max()) + 1)
    return ids, counts
