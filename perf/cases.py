"""Performance cases of the GSL-LPA library: what a program has it do, end to end.

Every case is one kind of call on one kind of graph:

  op       lpa       gsl_lpa on one graph (weights uint32 or none)
           noalloc   gsl_lpa_noalloc, the call for code that must not allocate
           f32       gsl_lpa_f32, float weights summed in double
           batched   gsl_lpa_batched, a batch as one concatenated CSR
           graphs    gsl_lpa_graphs, a batch of separately held graphs
           session   Session.add / Session.step, graphs arriving between steps
           split     gsl_split on raw label-propagation labels
           quality   gsl_modularity and gsl_disconnected on such labels
  kind     planted   equal blocks, random pairs inside and across blocks
           rmat      R-MAT (0.57, 0.19, 0.19, 0.05), ids shuffled
           road      two nearest neighbours of random points in a square
  weights  0: none (every weight 1), 16: whole numbers from 1 to 16

The graphs are those of this repository's workloads (planted 10,000 vertices,
R-MAT up to scale 26, road 24 M, batches of 200 to 200,000 vertices), made here
on the GPU from a seed.  Sizes depend on the case alone, the edges (and
weights) on the seed.  Every call runs 20 sweeps at most
and the tolerance 0.05, as the workloads do.
"""
import math
import random

import numpy as np
import torch

import paper_2403_01261_amd as gsl

MAX_ITERS = 20
TOLERANCE = 0.05


def listed():
    return [
        # the smallest graph of the batch workload on its own: a call's fixed cost
        {"name": "lpa-planted-200", "op": "lpa", "kind": "planted", "n": 200, "blocks": 10, "degree": 12, "weights": 0},
        # the planted workload: an interactive call on a small graph
        {"name": "lpa-planted-10k", "op": "lpa", "kind": "planted", "n": 10000, "blocks": 100, "degree": 12, "weights": 0},
        # a mean graph of the batch workload in a loop that must not allocate
        {"name": "noalloc-planted-29k", "op": "noalloc", "kind": "planted", "n": 28901, "blocks": 50, "degree": 20,
         "weights": 0},
        # the largest graph of the batch workload, dense and weighted, of odd size
        {"name": "lpa-planted-200k-w", "op": "lpa", "kind": "planted", "n": 199999, "blocks": 500, "degree": 32,
         "weights": 16},
        # the weighted social-network workload
        {"name": "lpa-rmat-s22-w", "op": "lpa", "kind": "rmat", "scale": 22, "factor": 16, "weights": 16},
        # the web-scale workload (hubs, four thousand million entries)
        {"name": "lpa-rmat-s26", "op": "lpa", "kind": "rmat", "scale": 26, "factor": 32, "weights": 0},
        # the road workload: short rows, no hubs, all 20 sweeps
        {"name": "lpa-road-24m", "op": "lpa", "kind": "road", "n": 24000000, "weights": 0},
        # the paper's own precision: float weights summed in double
        {"name": "f32-rmat-s20", "op": "f32", "kind": "rmat", "scale": 20, "factor": 16, "weights": 0},
        # the batch workload, a quarter of its graphs in one call
        {"name": "batched-1024", "op": "batched", "graphs": 1024, "nmin": 200, "nmax": 200000, "sizes": 5, "weights": 0},
        # one batch of the slot server under load: graphs in buffers of their own
        {"name": "graphs-117", "op": "graphs", "graphs": 117, "nmin": 200, "nmax": 200000, "sizes": 7, "weights": 0},
        # the continuous server: graphs that arrive in four groups between steps
        {"name": "session-48", "op": "session", "graphs": 48, "nmin": 200, "nmax": 20000, "sizes": 9, "weights": 0},
        # what a user reports of raw labels: modularity, disconnected communities
        {"name": "quality-road-6m", "op": "quality", "kind": "road", "n": 6000000, "weights": 0},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["lpa", "lpa", "lpa", "noalloc", "f32", "batched", "graphs", "session", "split", "quality"])
    weights = 0 if op == "f32" else rng.choice([0, 16])
    if op == "batched":
        return {"op": op, "graphs": _log_uniform(rng, 8, 1024), "nmin": 200, "nmax": _log_uniform(rng, 2000, 200000),
                "sizes": rng.randrange(1000), "weights": weights}
    if op == "graphs":
        return {"op": op, "graphs": _log_uniform(rng, 2, 120), "nmin": 200, "nmax": _log_uniform(rng, 2000, 200000),
                "sizes": rng.randrange(1000), "weights": weights}
    if op == "session":
        return {"op": op, "graphs": rng.randint(4, 60), "nmin": 200, "nmax": _log_uniform(rng, 1000, 100000),
                "sizes": rng.randrange(1000), "weights": weights}
    kind = "planted" if op == "noalloc" else rng.choice(["planted", "rmat", "road"])
    if kind == "rmat":
        return {"op": op, "kind": kind, "scale": rng.randint(8, 24), "factor": rng.randint(4, 32), "weights": weights}
    if kind == "road":
        return {"op": op, "kind": kind, "n": _log_uniform(rng, 1000, 20000000), "weights": weights}
    n = _log_uniform(rng, 200, 500000 if op == "noalloc" else 2000000)
    return {"op": op, "kind": kind, "n": n, "blocks": max(1, min(_log_uniform(rng, 5, 500), n // 10)),
            "degree": rng.randint(6, 32), "weights": weights}


# ---------------------------------------------------------------------------
# graphs
# ---------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _rand(g, n):
    return torch.rand(n, generator=g, device="cuda", dtype=torch.float64)


def _csr(parts, n, bits):
    """Symmetric CSR of the pairs (u << bits | v) in a list of tensors, both directions, without self loops and
    repeats.  Large graphs are sorted one range of rows after another."""
    mask = (1 << bits) - 1
    ranges = max(1, 2 * sum(p.numel() for p in parts) >> 29)
    ends = [n * k // ranges for k in range(ranges + 1)]
    off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    cols = []
    for lo, hi in zip(ends, ends[1:]):
        both = []
        for p in parts:
            u, v = p >> bits, p & mask
            other = u != v
            both.append(p[other & (u >= lo) & (u < hi)] if ranges > 1 else p[other])
            p = (v << bits) | u
            both.append(p[other & (v >= lo) & (v < hi)] if ranges > 1 else p[other])
        both = torch.unique(torch.cat(both))
        off[lo + 1:hi + 1] = torch.bincount((both >> bits) - lo, minlength=hi - lo)
        cols.append((both & mask).to(torch.int32))
        del both
    off = torch.cumsum(off, 0)
    return off, cols[0] if ranges == 1 else torch.cat(cols)


def _rmat(scale, factor, g):
    n, m, chunk = 1 << scale, factor << scale, 1 << 26
    a, ab, abc = 0.57, 0.76, 0.95
    perm = torch.randperm(n, generator=g, device="cuda")
    parts = []
    for lo in range(0, m, chunk):
        k = min(chunk, m - lo)
        u = torch.zeros(k, dtype=torch.int32, device="cuda")
        v = torch.zeros(k, dtype=torch.int32, device="cuda")
        for _ in range(scale):
            r = torch.rand(k, generator=g, device="cuda")
            low = r >= ab
            u.mul_(2).add_(low)
            v.mul_(2).add_((r >= a) ^ low ^ (r >= abc))
        parts.append((perm[u] << scale) | perm[v])
    return _csr(parts, n, scale)


def _planted_pairs(base, n, blocks, degree, g):
    """Pairs of planted graphs laid end to end: arrays (one value a graph) of first vertex, vertices, blocks, degree."""
    which = torch.arange(n.numel(), device="cuda")
    inside = torch.repeat_interleave(which, (n * (degree - 2) / 2).round().to(torch.int64))
    x = (_rand(g, inside.numel()) * n[inside]).to(torch.int64)
    b = x * blocks[inside] // n[inside]
    lo = -(-b * n[inside] // blocks[inside])
    hi = -(-(b + 1) * n[inside] // blocks[inside])
    y = lo + (_rand(g, x.numel()) * (hi - lo)).to(torch.int64)
    x, y = x + base[inside], y + base[inside]
    across = torch.repeat_interleave(which, n)
    s = (_rand(g, across.numel()) * n[across]).to(torch.int64) + base[across]
    t = (_rand(g, across.numel()) * n[across]).to(torch.int64) + base[across]
    return torch.cat([x, s]), torch.cat([y, t])


def _planted(n, blocks, degree, g):
    one = lambda x: torch.tensor([x], dtype=torch.int64, device="cuda")  # noqa: E731
    u, v = _planted_pairs(one(0), one(n), one(blocks), one(degree), g)
    bits = max(1, (n - 1).bit_length())
    return _csr([(u << bits) | v], n, bits)


def _road(n, g):
    """Two nearest neighbours of every point among the 3 x 3 cells around it, in either direction."""
    side = max(1, int(math.sqrt(n / 2)))
    x, y = torch.rand(n, generator=g, device="cuda"), torch.rand(n, generator=g, device="cuda")
    cell = (y * side).long().clamp_(max=side - 1) * side + (x * side).long().clamp_(max=side - 1)
    cell, order = torch.sort(cell)
    x, y = x[order], y[order]
    start = torch.searchsorted(cell, torch.arange(side * side + 1, device="cuda"))
    cx, cy = cell % side, cell // side
    here = torch.arange(n, device="cuda")
    best = [torch.full((n,), math.inf, device="cuda") for _ in range(2)]
    near = [here.clone() for _ in range(2)]
    for dy in (-1, 0, 1):
        row = cy + dy
        ok = (row >= 0) & (row < side)
        row = row.clamp_(0, side - 1)
        lo = start[row * side + (cx - 1).clamp_(min=0)]
        hi = torch.where(ok, start[row * side + (cx + 1).clamp_(max=side - 1) + 1], lo)
        for j in range(int((hi - lo).max())):
            p = lo + j
            other = (p < hi) & (p != here)
            p = torch.where(other, p, here)
            d = torch.where(other, (x[p] - x) ** 2 + (y[p] - y) ** 2, math.inf)
            first, second = d < best[0], d < best[1]
            near[1] = torch.where(first, near[0], torch.where(second, p, near[1]))
            best[1] = torch.where(first, best[0], torch.where(second, d, best[1]))
            near[0] = torch.where(first, p, near[0])
            best[0] = torch.where(first, d, best[0])
    bits = max(1, (n - 1).bit_length())
    return _csr([(order << bits) | order[q] for q in near], n, bits)


def _hash_of_pairs(off, cols, seed):
    """A 31-bit number for each entry, the same for (u, v) and (v, u)."""
    n = off.numel() - 1
    rows = torch.repeat_interleave(torch.arange(n, dtype=torch.int32, device="cuda"), off[1:] - off[:-1])
    h = torch.minimum(rows, cols).long() * 1000003 + torch.maximum(rows, cols)
    del rows
    h = (h ^ (seed * 7919)) * 0x9E3779B97F4A7C1
    h = (h ^ (h >> 29)) * 0x2545F4914F6CDD1D
    return (h >> 33) & 0x7FFFFFFF


def _weights(off, cols, most, seed):
    if not most:
        return None
    return (_hash_of_pairs(off, cols, seed) % most + 1).to(torch.int32)


def _graph(case, seed):
    g = _generator(seed)
    if case["kind"] == "rmat":
        off, cols = _rmat(case["scale"], case["factor"], g)
    elif case["kind"] == "road":
        off, cols = _road(case["n"], g)
    else:
        off, cols = _planted(case["n"], case["blocks"], case["degree"], g)
    return off, cols, _weights(off, cols, case["weights"], seed)


def _batch_sizes(case):
    """(vertices, blocks, mean degree) of every graph of a batch."""
    rng = random.Random(case["sizes"])
    out = []
    for _ in range(case["graphs"]):
        n = _log_uniform(rng, case["nmin"], case["nmax"])
        out.append((n, max(1, min(_log_uniform(rng, 5, 500), n // 10)), rng.randint(8, 32)))
    return out


def _batch(case, seed):
    """A batch as (first vertices, first entries, offsets, columns in local ids, weights)."""
    g = _generator(seed)
    n, blocks, degree = (torch.tensor(x, dtype=torch.int64, device="cuda") for x in zip(*_batch_sizes(case)))
    base = torch.zeros(n.numel() + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(n, 0, out=base[1:])
    total = int(base[-1])
    u, v = _planted_pairs(base[:-1], n, blocks, degree, g)
    bits = max(1, (total - 1).bit_length())
    off, cols = _csr([(u << bits) | v], total, bits)
    w = _weights(off, cols, case["weights"], seed)
    edge_base = off[base]
    first = torch.repeat_interleave(base[:-1], edge_base[1:] - edge_base[:-1])
    return base, edge_base.contiguous(), off, (cols - first).to(torch.int32), w


def _separate(case, seed):
    """The batch's graphs, each in arrays of its own, and the labels they share one buffer for."""
    base, edge_base, off, cols, w = _batch(case, seed)
    vb, eb = base.tolist(), edge_base.tolist()
    labels = torch.empty(vb[-1], dtype=torch.int32, device="cuda")
    out = []
    for k in range(case["graphs"]):
        e = slice(eb[k], eb[k + 1])
        out.append((off[vb[k]:vb[k + 1] + 1] - eb[k], cols[e].clone(), None if w is None else w[e].clone(),
                    labels[vb[k]:vb[k + 1]]))
    return out, labels


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------

def prepare(case, seed):
    gsl.load()
    op = case["op"]
    state = {"op": op}
    if op == "batched":
        state["batch"] = _batch(case, seed)
        state["out"] = torch.empty(state["batch"][2].numel() - 1, dtype=torch.int32, device="cuda")
        return state
    if op in ("graphs", "session"):
        state["graphs"], state["out"] = _separate(case, seed)
        if op == "session":
            v = sum(x[0].numel() - 1 for x in state["graphs"])
            e = sum(x[1].numel() for x in state["graphs"])
            state["session"] = gsl.Session(v, max(e, 1), max_graphs=64, max_iters=MAX_ITERS, tolerance=TOLERANCE,
                                           weighted=bool(case["weights"]))
        return state
    off, cols, w = _graph(case, seed)
    if op == "f32":
        w = ((_hash_of_pairs(off, cols, seed) >> 7) + 1).to(torch.float32) / float(1 << 24)
    state["graph"] = (off, cols, w)
    if op in ("split", "quality"):
        state["labels"] = gsl.gsl_lpa_ex(off, cols, w, MAX_ITERS, TOLERANCE, split=False)[0]
    if op != "quality":
        state["out"] = torch.empty(off.numel() - 1, dtype=torch.int32, device="cuda")
    return state


def _serve(session, graphs):
    """Four groups of graphs join a session, one group before each step; steps of at most 16 sweeps until all are done."""
    sweeps, running, arrived = [0] * len(graphs), {}, 0
    group = -(-len(graphs) // 4)
    while arrived < len(graphs) or running:
        if arrived < len(graphs):
            want = graphs[arrived:arrived + group]
            for k, (ticket, status, _) in enumerate(session.add(want)):
                if status != gsl.GSL_OK:
                    break
                running[ticket] = arrived + k
            else:
                k += 1
            arrived += k
        for ticket, ran in session.step(16):
            sweeps[running.pop(ticket)] = ran
    return np.array(sweeps, dtype=np.int32)


def run(state):
    op = state["op"]
    if op == "batched":
        base, edge_base, off, cols, w = state["batch"]
        labels, sweeps, _ = gsl.gsl_lpa_batched(base, edge_base, off, cols, w, MAX_ITERS, TOLERANCE, out=state["out"])
        return {"labels": labels, "sweeps": sweeps}
    if op == "graphs":
        _, sweeps, _ = gsl.gsl_lpa_graphs(state["graphs"], MAX_ITERS, TOLERANCE)
        return {"labels": state["out"], "sweeps": np.array(sweeps, dtype=np.int32)}
    if op == "session":
        sweeps = _serve(state["session"], state["graphs"])
        return {"labels": state["out"], "sweeps": sweeps}
    off, cols, w = state["graph"]
    if op == "lpa":
        return gsl.gsl_lpa(off, cols, w, MAX_ITERS, TOLERANCE, out=state["out"])
    if op == "noalloc":
        return gsl.gsl_lpa_noalloc(off, cols, w, MAX_ITERS, TOLERANCE, out=state["out"])
    if op == "f32":
        return gsl.gsl_lpa_f32(off, cols, w, MAX_ITERS, TOLERANCE, out=state["out"])[0]
    if op == "split":
        return gsl.gsl_split(off, cols, state["labels"], out=state["out"])
    q = gsl.gsl_modularity(off, cols, w, state["labels"])
    count, flags = gsl.gsl_disconnected(off, cols, state["labels"])
    return {"q": q, "disconnected": count, "flags": flags}


def work(case):
    """Offsets, columns and weights read once, labels written once.  The entries left after removing repeats are
    estimated (R-MAT keeps about 96 % of its edges, a road vertex has 2.58 neighbours)."""
    if "graphs" in case:
        sizes = _batch_sizes(case)
        n = sum(s[0] for s in sizes)
        nnz = sum(s[0] * s[2] for s in sizes)
    elif case["kind"] == "rmat":
        n = 1 << case["scale"]
        nnz = int(2 * 0.96 * n * case["factor"])
    elif case["kind"] == "road":
        n, nnz = case["n"], int(2.58 * case["n"])
    else:
        n, nnz = case["n"], case["n"] * case["degree"]
    entry = 8 if case["weights"] or case["op"] == "f32" else 4
    once = 8 * (n + 1) + entry * nnz + 4 * n
    if case["op"] == "split":
        return {"bytes": 8 * (n + 1) + 4 * nnz + 8 * n, "flops": 0}
    if case["op"] == "quality":
        return {"bytes": once + 8 * (n + 1) + 4 * nnz + 5 * n, "flops": 0}
    return {"bytes": once, "flops": 0}


def exact(case, seed):
    """The modularity; everything else a case returns is whole numbers."""
    if case["op"] != "quality":
        return None
    state = prepare(case, seed)
    off, cols, w = state["graph"]
    c = state["labels"].long()
    rows = torch.repeat_interleave(torch.arange(c.numel(), device="cuda"), off[1:] - off[:-1])
    w = torch.ones_like(cols, dtype=torch.int64) if w is None else w.long()
    total = int(w.sum())
    if total == 0:
        return {"q": 0.0, "disconnected": None, "flags": None}
    inside = int(w[c[rows] == c[cols.long()]].sum())
    strength = torch.zeros(c.numel(), dtype=torch.int64, device="cuda").index_add_(0, c[rows], w)
    return {"q": inside / total - float(((strength.double() / total) ** 2).sum()), "disconnected": None, "flags": None}
