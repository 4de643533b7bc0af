"""The work this library is used for, as cases that can be timed and compared.

A case is one call (or one group of calls) of a program that keeps its graph
uploaded: SSSP, BFS or CC from a seeded source, a minimum spanning forest, the
three traversals of one graph in flight together, a batch of small instances,
or a burst of queries to the serving loop.  Graphs are made on the GPU from
the seed alone, in the three shapes the library's own workloads have (R-MAT,
uniform, grid with shortcuts), and uploaded from host arrays as a program
that read them from a file would.
"""
from __future__ import annotations

import math
import random
import time

import numpy as np
import torch

from paper_1903_01665_amd import gen, gg

INF = 2**31 - 1
RMAT = (0.57, 0.19, 0.19)
VARIANTS = {"auto": (gg.MODE_AUTO, gg.SCHED_AUTO),
            "vertex-sync": (gg.VERTEX, gg.SYNC), "vertex-async": (gg.VERTEX, gg.ASYNC),
            "edge-sync": (gg.EDGE, gg.SYNC), "edge-async": (gg.EDGE, gg.ASYNC)}


def single(name, kind, family, n, m, variant="auto"):
    """One R-MAT or uniform graph: kind is sssp, bfs, cc, msf or step."""
    return {"name": name, "kind": kind, "family": family, "n": n, "m": m, "variant": variant}


def lattice(name, kind, width, height):
    return {"name": name, "kind": kind, "family": "grid", "width": width, "height": height,
            "variant": "auto"}


def many(name, kind, count, graphs, lo, hi):
    """batch: `count` instances, each with a graph of its own; serve: `count`
    queries over `graphs` resident graphs.  R-MAT scales lo..hi."""
    return {"name": name, "kind": kind, "family": "rmat", "count": count, "graphs": graphs,
            "lo": lo, "hi": hi}


def listed():
    return [
        # the smallest graph a query or a batch instance has: one call is latency
        single("bfs-rmat10", "bfs", "rmat", 1 << 10, 16 << 10),
        # the small uniform workload graph
        single("sssp-er16k", "sssp", "uniform", 16384, 131072),
        # a program that picks the schedule itself: the plain vertex worklist
        single("sssp-rmat18-worklist", "sssp", "rmat", 1 << 18, 16 << 18, "vertex-async"),
        # a social graph whose sizes are no round numbers
        single("bfs-rmat-odd", "bfs", "rmat", 3000017, 30000001),
        # components of a sparse random graph, odd sizes
        single("cc-uniform-odd", "cc", "uniform", 1000003, 4000037),
        # a city-sized road network: deep, and narrow in every round
        lattice("sssp-grid-odd", "sssp", 1023, 777),
        # the benchmark's step: SSSP, BFS and CC of one skewed graph in flight together
        single("step-rmat22", "step", "rmat", 1 << 22, 16 << 22),
        # the same on the large uniform graph (random gathers without locality)
        single("step-er23", "step", "uniform", 1 << 23, 1 << 26),
        # shortest paths on the country-sized road network
        lattice("sssp-grid4096", "sssp", 4096, 4096),
        # spanning forest of a skewed graph
        single("msf-rmat20", "msf", "rmat", 1 << 20, 16 << 20),
        # many small independent instances in one launch sequence
        many("batch-48", "batch", 48, 48, 10, 17),
        # a burst of queries to the serving loop over resident graphs
        many("serve-48", "serve", 48, 4, 12, 19),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sssp", "sssp", "sssp", "bfs", "bfs", "cc", "cc", "msf", "step", "batch",
                       "serve"])
    if kind == "batch":
        lo = rng.randint(10, 13)
        n = _log(rng, 6, 48)
        c = many("", kind, n, n, lo, rng.randint(lo + 1, 17))
    elif kind == "serve":
        lo = rng.randint(10, 14)
        c = many("", kind, _log(rng, 6, 48), rng.randint(2, 4), lo, rng.randint(lo + 1, 19))
    else:
        # (the components of a grid are always one)
        family = rng.choice(["rmat", "uniform"] if kind in ("step", "cc") else
                            ["rmat", "uniform", "grid"])
        if family == "grid":
            w = _log(rng, 32, 4096)
            c = lattice("", kind, w, max(32, int(w * rng.uniform(0.5, 1.0))))
        else:
            n = _log(rng, 1 << 10, 1 << 22 if family == "rmat" else 1 << 23)
            # sparse uniform graphs have several components, dense ones do not
            deg = rng.uniform(8, 32) if family == "rmat" else \
                rng.uniform(0.7, 2.5) if kind == "cc" else rng.uniform(4, 16)
            m = min(int(n * deg), 1 << 24 if kind == "msf" else 1 << 26)
            c = single("", kind, family, n, m)
            if kind in ("sssp", "bfs") and m <= 1 << 23 and rng.random() < 0.3:
                c["variant"] = rng.choice([v for v in VARIANTS if v != "auto"])
    del c["name"]
    return c


# ------------------------------------------------------------------ graphs --
def _generator(*key):
    g = torch.Generator(device="cuda")
    g.manual_seed(random.Random(repr(key)).randrange(1 << 62))
    return g


def _rmat(n, m, g):
    """Recursive R-MAT: a quadrant of the adjacency matrix per bit; a vertex
    count that is no power of two scales the ids down."""
    a, b, c = RMAT
    src = torch.zeros(m, dtype=torch.int32, device="cuda")
    dst = torch.zeros(m, dtype=torch.int32, device="cuda")
    scale = max(1, (n - 1).bit_length())
    for _ in range(scale):
        r = torch.rand(m, generator=g, device="cuda")
        low = r >= a + b
        src.mul_(2).add_(low)
        dst.mul_(2).add_(torch.where(low, r >= a + b + c, r >= a))
    if n != 1 << scale:
        src = ((src.long() * n) >> scale).int()
        dst = ((dst.long() * n) >> scale).int()
    return src, dst


def _uniform(n, m, g):
    src = torch.randint(0, n, (m,), generator=g, device="cuda", dtype=torch.int32)
    dst = torch.randint(0, n, (m,), generator=g, device="cuda", dtype=torch.int32)
    return src, torch.where(dst == src, (dst + 1) % n, dst)


def _grid(width, height, g):
    """4-neighbour grid with 1% of its edges again as shortcuts of span <= 8;
    both directions of an edge share a weight."""
    ids = torch.arange(width * height, dtype=torch.int32, device="cuda").view(height, width)
    count = (width * (height - 1) + height * (width - 1)) // 100
    x = torch.randint(0, width, (count,), generator=g, device="cuda")
    y = torch.randint(0, height, (count,), generator=g, device="cuda")
    dx = torch.randint(-8, 9, (count,), generator=g, device="cuda")
    dy = torch.randint(-8, 9, (count,), generator=g, device="cuda")
    keep = (dx.abs() + dy.abs() >= 2) & (x + dx >= 0) & (x + dx < width) & (y + dy >= 0) & \
        (y + dy < height)
    a = (y * width + x)[keep].int()
    b = ((y + dy) * width + x + dx)[keep].int()
    src = torch.cat([ids[:, :-1].reshape(-1), ids[:-1].reshape(-1), a])
    dst = torch.cat([ids[:, 1:].reshape(-1), ids[1:].reshape(-1), b])
    w = torch.randint(1, 1001, (src.numel(),), generator=g, device="cuda", dtype=torch.int32)
    return torch.cat([src, dst]), torch.cat([dst, src]), torch.cat([w, w])


def _edges(case, seed):
    """(n, src, dst, w) on the GPU, sorted by source, generation order kept in a row."""
    g = _generator(case["family"], seed)
    if case["family"] == "grid":
        n = case["width"] * case["height"]
        src, dst, w = _grid(case["width"], case["height"], g)
    else:
        n = case["n"]
        src, dst = (_rmat if case["family"] == "rmat" else _uniform)(n, case["m"], g)
        w = torch.randint(1, 101, (case["m"],), generator=g, device="cuda", dtype=torch.int32)
    src, order = torch.sort(src, stable=True)
    return n, src, dst[order], w[order]


def _host(case, seed):
    n, src, dst, w = _edges(case, seed)
    row = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    row[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0)
    h = [x.to(torch.int32).cpu().numpy() for x in (row, dst, w)]
    return gen.HostGraph(n, *h, symmetric=case["family"] == "grid")


def _source(hg, seed):
    """A vertex with an out-edge."""
    rng = random.Random("source %d" % seed)
    while True:
        v = rng.randrange(hg.n)
        if hg.row_ptr[v + 1] > hg.row_ptr[v]:
            return v


def _members(case):
    """Graphs of a batch or a server, and its queries as (graph, algo): the
    sizes come from the case, the edges from the seed."""
    rng = random.Random(repr(sorted((k, v) for k, v in case.items() if k != "name")))
    graphs = []
    for _ in range(case["graphs"]):
        s = rng.randint(case["lo"], case["hi"])
        ef = rng.randint(8, 32) if case["kind"] == "batch" else 16
        graphs.append({"family": "rmat", "n": 1 << s, "m": ef << s})
    if case["kind"] == "batch":
        return graphs, [(i, rng.randint(0, 1)) for i in range(case["count"])]
    return graphs, [(rng.randrange(case["graphs"]), rng.randint(0, 1))
                    for _ in range(case["count"])]


# ------------------------------------------------------------------- calls --
class State:
    """What a program keeps between calls; gives the handles back at its end."""

    def __init__(self):
        self.workspaces, self.graph, self.batch, self.server = [], None, None, None

    def __del__(self):
        torch.cuda.synchronize()
        for x in [*self.workspaces, self.graph, self.batch, self.server]:
            if x is not None:
                x.free()


def _int32(n):
    return torch.empty(n, dtype=torch.int32, device="cuda")


def prepare(case, seed):
    s = State()
    s.kind = kind = case["kind"]
    if kind in ("batch", "serve"):
        graphs, queries = _members(case)
        hosts = [_host(g, seed * 1000 + i) for i, g in enumerate(graphs)]
        sources = [_source(hosts[g], seed * 1000 + i) for i, (g, _) in enumerate(queries)]
        if kind == "batch":
            s.batch = gg.Batch([(a, hosts[g], v) for (g, a), v in zip(queries, sources)])
            s.out = _int32(s.batch.total_n)
            s.views = [s.out[o:o + hosts[g].n] for o, (g, _) in
                       zip(s.batch.offsets().tolist(), queries)]
        else:
            s.server = gg.Server(slots=8)
            ids = [s.server.add_graph(gg.Graph.from_host(h, symmetrize=True)) for h in hosts]
            s.queries = [(ids[g], a, v, _int32(hosts[g].n)) for (g, a), v in
                         zip(queries, sources)]
        return s
    hg = _host(case, seed)
    s.graph = gg.Graph.from_host(hg, symmetrize=kind in ("bfs", "cc", "step"))
    s.graph.probe()
    s.source = _source(hg, seed)
    s.variant = VARIANTS[case["variant"]]
    if kind == "step":
        s.workspaces = [gg.Workspace(s.graph) for _ in range(3)]
    if kind == "msf":
        s.out = torch.empty(hg.m, dtype=torch.uint8, device="cuda")
    else:
        s.out = [_int32(hg.n) for _ in range(3 if kind == "step" else 1)]
    return s


def run(s):
    if s.kind == "sssp":
        return s.graph.sssp(s.source, *s.variant, out=s.out[0])
    if s.kind == "bfs":
        return s.graph.bfs(s.source, *s.variant, out=s.out[0])
    if s.kind == "cc":
        return s.graph.cc(*s.variant, out=s.out[0])
    if s.kind == "msf":
        return s.graph.msf(out=s.out)
    if s.kind == "step":
        ws = s.workspaces
        tickets = [s.graph.sssp_async(s.source, out=s.out[0], ws=ws[0]),
                   s.graph.bfs_async(s.source, out=s.out[1], ws=ws[1]),
                   s.graph.cc_async(out=s.out[2], ws=ws[2])]
        out = [t.wait() for t in tickets]
        for t in tickets:
            t.free()
        return out
    if s.kind == "batch":
        s.batch.run(out=s.out)
        return s.views
    for gid, algo, source, out in s.queries:
        s.server.submit(gid, algo, source, out)
    left = len(s.queries)
    while left:
        done = s.server.poll()
        if any(d[1] != 0 for d in done):
            raise RuntimeError("a query failed: %r" % done)
        left -= len(done)
        if left:
            time.sleep(2e-5)
    return [q[3] for q in s.queries]


# ------------------------------------------------------- work and results --
def _one(kind, n, m):
    """Each array once: offsets, columns (and weights), the result."""
    if kind == "step":
        parts = [_one(k, n, m) for k in ("sssp", "bfs", "cc")]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    edge = {"sssp": 8, "bfs": 4, "cc": 4, "msf": 9}[kind]
    return {"bytes": 4 * (n + 1) + edge * m + (0 if kind == "msf" else 4 * n), "flops": m}


def work(case):
    kind = case["kind"]
    if kind in ("batch", "serve"):
        graphs, queries = _members(case)
        parts = [_one(("sssp", "bfs")[a], graphs[g]["n"], graphs[g]["m"]) for g, a in queries]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    if case["family"] == "grid":
        w, h = case["width"], case["height"]
        half = w * (h - 1) + h * (w - 1)
        return _one(kind, w * h, 2 * (half + half // 100))
    return _one(kind, case["n"], case["m"])


def _paths(n, src, dst, w, source):
    """Relax every edge until nothing changes (w None: one per edge)."""
    dist = torch.full((n,), INF, dtype=torch.int64, device="cuda")
    dist[source] = 0
    src, dst = src.long(), dst.long()
    while True:
        du = dist[src]
        cand = torch.where(du < INF, du + (1 if w is None else w), INF).clamp_(max=INF)
        new = dist.scatter_reduce(0, dst, cand, "amin")
        if torch.equal(new, dist):
            return dist
        dist = new


def _flatten(parent):
    while True:
        up = parent[parent]
        if torch.equal(up, parent):
            return parent
        parent = up


def _labels(n, src, dst):
    """Smallest id of each component: hang roots under smaller ones."""
    parent = torch.arange(n, device="cuda")
    src, dst = src.long(), dst.long()
    while True:
        a, b = parent[src], parent[dst]
        if torch.equal(a, b):
            return parent
        hooked = parent.scatter_reduce(0, torch.maximum(a, b), torch.minimum(a, b), "amin")
        parent = _flatten(hooked)


def _forest(n, src, dst, w):
    """Boruvka with the keys (weight, edge index)."""
    m = src.numel()
    top = torch.iinfo(torch.int64).max
    comp = torch.arange(n, device="cuda")
    chosen = torch.zeros(m, dtype=torch.uint8, device="cuda")
    key = (w.long() << 32) | torch.arange(m, device="cuda")
    src, dst = src.long(), dst.long()
    while True:
        a, b = comp[src], comp[dst]
        cross = a != b
        if not bool(cross.any()):
            break
        k = torch.where(cross, key, top)
        best = torch.full((n,), top, dtype=torch.int64, device="cuda")
        best = best.scatter_reduce(0, a, k, "amin").scatter_reduce(0, b, k, "amin")
        roots = torch.nonzero(best < top).view(-1)
        e = best[roots] & 0xffffffff
        chosen[e] = 1
        parent = torch.arange(n, device="cuda")
        parent[roots] = a[e] + b[e] - roots
        twice = parent[parent] == torch.arange(n, device="cuda")  # both ends chose one edge
        parent = torch.where(twice & (torch.arange(n, device="cuda") < parent),
                             torch.arange(n, device="cuda"), parent)
        comp = _flatten(parent)[comp]
    picked = chosen.bool()
    return [chosen, int(w[picked].sum(dtype=torch.int64)), int(picked.sum())]


def exact(case, seed):
    kind = case["kind"]
    if kind in ("batch", "serve"):
        graphs, queries = _members(case)
        out = []
        for i, (g, algo) in enumerate(queries):
            at = seed * 1000 + g
            n, src, dst, w = _edges(graphs[g], at)
            v = _source(_host(graphs[g], at), seed * 1000 + i)
            out.append(_paths(n, src, dst, w if algo == 0 else None, v))
        return out
    if case["family"] == "grid" and kind in ("sssp", "bfs") and case["width"] > 1200:
        return None  # thousands of sweeps over tens of millions of edges
    n, src, dst, w = _edges(case, seed)
    if kind == "msf":
        return _forest(n, src, dst, w)
    if kind == "cc":
        return _labels(n, src, dst)
    v = _source(_host(case, seed), seed)
    if kind == "step":
        return [_paths(n, src, dst, w, v), _paths(n, src, dst, None, v), _labels(n, src, dst)]
    return _paths(n, src, dst, w if kind == "sssp" else None, v)
