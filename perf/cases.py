"""Traversal workloads that a user of the library has it do, for measuring it.

A case is one call on one graph handle: an algorithm, a synthetic graph (R-MAT or uniform
random), how much of its edge data the device budget holds, and for batched calls the number
of sources.  `prepare` builds the graph and the handle, `run` makes the call through the
public Python entry points, `exact` computes PageRank's and personalized PageRank's values in
64 bits with plain torch.

Ranges: 2^10 to 2^24 vertices (powers of two and odd counts), 4 to 32 edge samples per vertex,
everything resident (the library's default budget) or a device budget of a quarter to a
half of the edge bytes, 1 to 64 sources per batched call.
"""
import math

import numpy as np
import torch

import paper_2208_14935_amd as hy

# R-MAT quadrants of every synthetic graph of this repository
A, B, C = 0.57, 0.19, 0.19
PR_STEPS, PPR_STEPS, DAMPING = 20, 10, 0.85


def _case(algo, n, ef, graph="rmat", budget=0.0, lanes=0, pack=True, pinned=True, name=None):
    c = {"algo": algo, "n": n, "ef": ef, "graph": graph, "budget": budget, "lanes": lanes, "pack": pack,
         "pinned": pinned}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a query on a small graph: launches, synchronisations and host work per iteration
        _case("bfs", 1 << 10, 16, pinned=False, name="bfs-tiny"),
        # one traversal over a graph that fits the device (the default budget), result in pinned memory
        _case("bfs", 1 << 22, 16, name="bfs-resident"),
        # the hybrid engines: a quarter of the edges on the device, the rest over the host link
        _case("bfs", 1 << 23, 16, budget=0.25, name="bfs-budget"),
        # weighted graph on the device, weights packed into the edge words; an odd vertex count
        _case("sssp", 2_500_009, 16, name="sssp-resident"),
        # weights kept apart as bytes (what graphs of more than 2^26 vertices use), a quarter resident
        _case("sssp", 1 << 22, 16, budget=0.25, pack=False, name="sssp-budget"),
        # components of a uniform random graph with an odd vertex count: no hubs, long sparse tail
        _case("cc", 3_000_017, 8, graph="er", name="cc-resident"),
        # components of a skewed graph over the host link
        _case("cc", 1 << 21, 16, budget=0.25, name="cc-budget"),
        # ranks of the largest graph of the range, resident: 20 passes over 2.6e8 edges
        _case("pagerank", 1 << 24, 16, name="pagerank-resident"),
        # ranks over the host link
        _case("pagerank", 1 << 22, 16, budget=0.25, name="pagerank-budget"),
        # a full batch of sources served by one traversal, edges over the host link
        _case("bfs", 1 << 20, 16, budget=0.25, lanes=64, name="batch-bfs"),
        # a partly filled batch of weighted queries, as a query server steps it
        _case("sssp", 1 << 18, 16, lanes=37, name="batch-sssp"),
        # a full batch of personalized PageRank queries on a resident graph
        _case("ppr", 1 << 20, 16, lanes=64, name="batch-ppr"),
    ]


# kinds of call, with the edge samples of the largest drawn case of each
_KINDS = [("bfs", 0.0, 0, 1 << 27), ("bfs", 0.25, 0, 1 << 27), ("sssp", 0.0, 0, 1 << 26), ("sssp", 0.25, 0, 1 << 26),
          ("cc", 0.0, 0, 1 << 25), ("cc", 0.25, 0, 1 << 25), ("pagerank", 0.0, 0, 1 << 27),
          ("pagerank", 0.25, 0, 1 << 26), ("bfs", 0.25, 1, 1 << 24), ("sssp", 0.0, 1, 1 << 23), ("ppr", 0.0, 1, 1 << 23)]


def draw(rng):
    algo, budget, batch, most = rng.choice(_KINDS)
    ef = rng.choice([4, 7, 8, 12, 16, 24, 32])
    n = int(round(2.0 ** rng.uniform(10, math.log2(most // ef))))
    if rng.random() < 0.5:
        n |= 1
    if budget:
        n = max(n, 1 << 17)
        budget = rng.choice([0.25, 0.35, 0.5])
    lanes = int(round(2.0 ** rng.uniform(0, 6))) if batch else 0
    return _case(algo, n, ef, graph=rng.choice(["rmat", "rmat", "er"]), budget=budget, lanes=lanes,
                 pack=rng.random() < 0.7, pinned=rng.random() < 0.8)


def _graph(case, seed):
    """Sorted CSR (offsets, neighbours) on the device: seeded samples, self-loops and duplicates
    removed; components run on the symmetrized graph."""
    n, m = case["n"], case["n"] * case["ef"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1_000_003 * seed + 17)
    if case["graph"] == "er":
        u = torch.randint(0, n, (m,), generator=gen, device="cuda")
        v = torch.randint(0, n, (m,), generator=gen, device="cuda")
    else:
        u = torch.zeros(m, dtype=torch.int32, device="cuda")
        v = torch.zeros(m, dtype=torch.int32, device="cuda")
        r = torch.empty(m, dtype=torch.float32, device="cuda")
        for _ in range((n - 1).bit_length()):
            r.uniform_(generator=gen)
            u.mul_(2).add_(r >= A + B)
            v.mul_(2).add_(((r >= A) & (r < A + B)) | (r >= A + B + C))
        u, v = u.long() % n, v.long() % n
    keep = u != v
    key = (u * n + v)[keep]
    if case["algo"] == "cc":
        key = torch.cat([key, (v * n + u)[keep]])
    del u, v, keep
    key = torch.unique(key)
    off = torch.searchsorted(key, torch.arange(n + 1, device="cuda") * n)
    return off, key.remainder_(n).int()


def _host(t, dtype):
    return t.cpu().numpy().view(dtype)


def _sources(case, off, seed):
    """Distinct-ish seeded sources among the vertices with out-edges."""
    deg = off[1:] - off[:-1]
    some = torch.nonzero(deg > 0).flatten()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2_000_003 * seed + 29)
    pick = torch.randint(0, some.numel(), (max(case["lanes"], 1),), generator=gen, device="cuda")
    return some[pick].cpu().numpy().astype(np.uint32)


def prepare(case, seed):
    off, col = _graph(case, seed)
    sources = _sources(case, off, seed)
    weights = None
    if case["algo"] == "sssp":
        gen = torch.Generator(device="cuda")
        gen.manual_seed(3_000_017 * seed + 41)
        w = torch.randint(1, 65, (col.numel(),), generator=gen, device="cuda", dtype=torch.int32)
        weights = _host(w, np.uint32)
        del w
    off, col = _host(off, np.uint64), _host(col, np.uint32)
    torch.cuda.empty_cache()
    g = hy.Graph(off, col, weights=weights, symmetric=case["algo"] == "cc", pack=case["pack"])
    if case["budget"]:
        # the calibrated cost model that the benchmark uses on these hosts
        g.set_params(gamma=(1, 1), rq_distinct_lines=1, zc_tie=2)
        g.set_budget(int(case["budget"] * g.edge_bytes(case["algo"]) * g.m))
    out = None
    if case["pinned"]:
        rows = max(case["lanes"], 1)
        out = hy.pinned_empty((rows, case["n"]), np.float32 if case["algo"] in ("pagerank", "ppr") else np.uint32)
    return {"graph": g, "algo": case["algo"], "lanes": case["lanes"], "sources": sources, "out": out}


def run(state):
    g, algo, out = state["graph"], state["algo"], state["out"]
    if state["lanes"]:
        values, iterations, _ = g.run_batch(algo, state["sources"], out=out)
    else:
        res = g.run(algo, int(state["sources"][0]), out=out)
        values, iterations = res.values, res.iterations
    if algo in ("pagerank", "ppr"):
        return {"values": values}
    # levels, distances and labels; only BFS pins its iteration count (a vertex may push a value
    # that improved within the iteration in the others)
    got = {"values": values.view(np.int32)}
    if algo == "bfs":
        got["iterations"] = np.asarray(iterations, dtype=np.int64)
    return got


def work(case):
    n, m, rows = case["n"], case["n"] * case["ef"], max(case["lanes"], 1)
    if case["algo"] == "cc":
        m *= 2
    d1 = 4 if case["algo"] != "sssp" or case["pack"] else 5
    if case["algo"] in ("pagerank", "ppr"):
        # every step reads every edge (and, batched, a value row of its source) and every vertex's
        # offset, and reads and writes every value
        steps = PR_STEPS if case["algo"] == "pagerank" else PPR_STEPS
        return {"bytes": steps * (4.0 * m + 8.0 * n + 8.0 * n * rows) + 4.0 * n * rows, "flops": 2.0 * steps * m * rows}
    return {"bytes": 1.0 * d1 * m + 8.0 * n + 4.0 * n * rows, "flops": 1.0 * m * rows}


def tolerance(case):
    # 32-bit values and shares; sums of up to 1e5 terms in an order that changes from run to run
    if case["algo"] == "pagerank":
        return {"rel": 1e-5, "max": 1e-3}
    if case["algo"] == "ppr":
        return {"rel": 1e-6, "max": 1e-5}
    return "exact"


def exact(case, seed):
    if case["algo"] not in ("pagerank", "ppr"):
        return None
    off, col = _graph(case, seed)
    n = case["n"]
    deg = off[1:] - off[:-1]
    src = torch.repeat_interleave(torch.arange(n, device="cuda", dtype=torch.int32), deg)
    inv = torch.where(deg > 0, 1.0 / deg.double(), torch.zeros(n, dtype=torch.float64, device="cuda"))
    if case["algo"] == "pagerank":
        x = torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
        for _ in range(PR_STEPS):
            y = torch.zeros(n, dtype=torch.float64, device="cuda")
            y.index_add_(0, col, (x * inv)[src])
            x = (1.0 - DAMPING) / n + DAMPING * y
        return {"values": x.cpu().numpy()}
    rows = []
    for s in _sources(case, off, seed).tolist():
        x = torch.zeros(n, dtype=torch.float64, device="cuda")
        x[s] = 1.0
        for _ in range(PPR_STEPS):
            y = torch.zeros(n, dtype=torch.float64, device="cuda")
            y.index_add_(0, col, (x * inv)[src])
            x = DAMPING * y
            x[s] += 1.0 - DAMPING
        rows.append(x.cpu().numpy())
    return {"values": np.stack(rows)}
