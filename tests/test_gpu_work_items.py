"""GPU parity where the work distribution changes with the graph's size: the
tiles of a frontier work item (1, 2 or 4 here) and the edges of a heavy-row
chunk (128, 256 or 512), with rows one edge below, at and above the chunk
sizes, in every schedule that uses them.
"""
import numpy as np
import pytest

import oracle
from paper_1903_01665_amd import gen

pytestmark = pytest.mark.gpu


def hub_graph(n, m, seed):
    """n vertices, m edges, most of them uniform; hub rows around the chunk sizes."""
    rng = np.random.default_rng(seed)
    lens = [127, 128, 129, 255, 256, 257, 511, 512, 513, 1025, 4097]
    hubs = rng.choice(n, size=len(lens), replace=False)
    src = np.concatenate([np.repeat(hubs, lens), rng.integers(0, n, m - sum(lens))])
    dst = rng.integers(0, n, m)
    dst[rng.integers(0, m, 64)] = hubs[0]
    return gen.from_edges(n, src, dst, rng.integers(1, 101, m), name=f"hub{n}"), int(hubs[-1])


@pytest.mark.parametrize("n,m", [(1048512, 2000003), (1048577, 4500001), (2097153, 8600003)])
def test_items_and_chunks(n, m):
    from paper_1903_01665_amd import gg
    hg, s = hub_graph(n, m, n)
    dist = oracle.sssp(hg.n, hg.row_ptr, hg.col, hg.w, s)
    lvl = oracle.bfs(hg.n, hg.row_ptr, hg.col, s)
    lab = oracle.cc(hg.n, hg.row_ptr, hg.col)
    for renumber in (False, True):
        g = gg.Graph.from_host(hg, symmetrize=True, transpose=True, renumber=renumber)
        try:
            for mode, sched, mapping, hops in ((0, gg.ASYNC, 3, 0), (0, gg.ASYNC, 3, 4),
                                               (0, gg.ASYNC, 1, 0), (1, gg.ASYNC, 0, 0),
                                               (0, gg.SYNC, 3, 0), (0, gg.DIROPT, 3, 0)):
                o = gg.make_opts(mode, sched, mapping, hops=hops)
                print(hg.name, renumber, mode, sched, mapping, hops, flush=True)
                np.testing.assert_array_equal(g.sssp(s, opts=o).cpu().numpy(), dist)
                np.testing.assert_array_equal(g.bfs(s, opts=o).cpu().numpy(), lvl)
                np.testing.assert_array_equal(g.cc(opts=o).cpu().numpy(), lab)
            nf = gg.make_opts(0, gg.NEARFAR, 3, hops=4, delta=60, far_degree=32)
            np.testing.assert_array_equal(g.sssp(s, opts=nf).cpu().numpy(), dist)
            cc = gg.make_opts(1, gg.DIROPT)
            np.testing.assert_array_equal(g.cc(opts=cc).cpu().numpy(), lab)
        finally:
            g.free()
