"""GPU parity of the traversals that run as one workgroup (small graphs, every
variant field left to the library) at the edges of their range: one vertex, a
vertex more than a bitmap word, rows around 16 and 64 edges, the most vertices
and edges, one more than that, values at and above INF, and the same through the batched,
served, host-asynchronous and allocation-free entry points.
"""
import ctypes

import numpy as np
import pytest

import oracle
from helpers import path_graph, random_graph, star
from paper_1903_01665_amd import gen

pytestmark = pytest.mark.gpu
INF = 2**31 - 1
LARGEST = 32768  # kSmallN


def row_lengths(lens, n):
    """Row v has lens[v % len(lens)] edges to consecutive heads."""
    src = np.repeat(np.arange(n), [lens[v % len(lens)] for v in range(n)])
    dst = (src * 7 + np.arange(len(src))) % n
    return gen.from_edges(n, src, dst, 1 + (np.arange(len(src)) * 37) % 101, name=f"rows{n}")


def graphs():
    rng = np.random.default_rng(20)
    heavy = random_graph(rng, 400, 3000, (1 << 30) - 4, (1 << 30) + 4, name="near-inf")
    return [gen.from_edges(1, [0], [0], [3], name="one"),
            gen.from_edges(33, [], [], [], name="empty33"),
            path_graph(1025, np.full(1024, 2**31 - 1 >> 9)),  # reaches INF on the way
            row_lengths([15, 16, 17, 63, 64, 65, 0, 1], 513), row_lengths([0, 300, 3], 97),
            star(31, [[9, 2]] * 31), heavy, gen.workload("rmat12"), gen.workload("grid63"),
            random_graph(rng, 5000, 32768, 1, 100, name="m32768"),
            random_graph(rng, 5000, 32769, 1, 100, name="m32769"),
            random_graph(rng, 5000, 65536, 1, 100, name="m65536"),
            random_graph(rng, 5000, 65537, 1, 100, name="m65537"),
            random_graph(rng, 20000, 131072, 1, 100, name="m131072"),
            random_graph(rng, 20000, 131073, 1, 100, name="m131073"),
            random_graph(rng, LARGEST - 1, 65535, 0, 100, name="n-1"),
            random_graph(rng, LARGEST, 40000, 1, 100, name="n"),
            random_graph(rng, LARGEST + 1, 60000, 1, 100, name="n+1")]


def expected(hg, s):
    return (oracle.sssp(hg.n, hg.row_ptr, hg.col, hg.w, s),
            oracle.bfs(hg.n, hg.row_ptr, hg.col, s), oracle.cc(hg.n, hg.row_ptr, hg.col))


@pytest.mark.parametrize("renumber", [None, True])
@pytest.mark.parametrize("hg", graphs(), ids=lambda h: h.name)
def test_whole_traversals(hg, renumber):
    import torch

    from paper_1903_01665_amd import gg
    g = gg.Graph.from_host(hg, renumber=renumber)
    try:
        for s in sorted({0, hg.n // 2, hg.n - 1}):
            print(hg.name, renumber, s, flush=True)
            d, b, c = expected(hg, s)
            for rep in range(2):
                np.testing.assert_array_equal(g.sssp(s).cpu().numpy(), d)
                np.testing.assert_array_equal(g.bfs(s).cpu().numpy(), b)
                np.testing.assert_array_equal(g.cc().cpu().numpy(), c)
            st = g.stats()
            assert st["rc"] == 0 and st["iterations"] >= 1
            t = [g.sssp_async(s), g.bfs_async(s, ws=(ws := gg.Workspace(g)))]
            np.testing.assert_array_equal(t[0].wait().cpu().numpy(), d)
            np.testing.assert_array_equal(t[1].wait().cpu().numpy(), b)
            [x.free() for x in t]
            ws.free()
            out = torch.full((hg.n,), -1, dtype=torch.int32, device="cuda")
            assert gg.lib().gg_bfs_noalloc(g.handle, s, None, ctypes.c_void_p(out.data_ptr()),
                                           gg._stream_ptr(None)) == 0
            np.testing.assert_array_equal(out.cpu().numpy(), b)
    finally:
        g.free()


def test_whole_batch_and_serving():
    import torch

    from paper_1903_01665_amd import gg
    hosts = graphs()
    inst = [(i % 2, h, h.n // 3) for i, h in enumerate(hosts + hosts[::-1])]
    want = [expected(h, s)[a] for a, h, s in inst]
    for flags in (0, gg.BATCH_NO_GRAPH, gg.BATCH_ONE_GROUP):
        b = gg.Batch(inst, flags=flags)
        try:
            out = torch.empty(b.total_n, dtype=torch.int32, device="cuda")
            for rep in range(3):
                out.fill_(-7)
                b.run(out)
                got = out.cpu().numpy()
                for o, (a, h, s), w in zip(b.offsets(), inst, want):
                    np.testing.assert_array_equal(got[o:o + h.n], w, err_msg=h.name)
        finally:
            b.free()
    srv = gg.Server(3)
    try:
        ids = [srv.add_graph(gg.Graph.from_host(h)) for h, in zip(h for _, h, _ in inst)]
        outs = [torch.full((h.n,), -7, dtype=torch.int32, device="cuda") for _, h, _ in inst]
        for (a, h, s), i, o in zip(inst, ids, outs):
            srv.submit(i, a, s, o)
        done = []
        while len(done) < len(inst):
            done += srv.poll()
        assert all(d[1] == 0 for d in done)
        torch.cuda.synchronize()
        for o, w in zip(outs, want):
            np.testing.assert_array_equal(o.cpu().numpy(), w)
    finally:
        srv.free()
