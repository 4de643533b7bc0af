"""GPU parity of CC by union-find where its passes change: neighbours per
vertex on both sides of the sparse and the dense rule, many components of
every size, chains and grids with and without the probe that finds them deep,
and graphs whose first neighbours say nothing (stars, cliques joined by one
late edge).
"""
import numpy as np
import pytest

import oracle
from helpers import path_graph, random_graph
from paper_1903_01665_amd import gen

pytestmark = pytest.mark.gpu


def shuffled_path(n, seed):
    p = np.random.default_rng(seed).permutation(n)
    return gen.from_edges(n, p[:-1], p[1:], np.ones(n - 1, np.int32), name=f"shuffled-path{n}")


def cliques(count, size):
    """`count` cliques, each joined to the next by the last edge of a row."""
    i, j = np.meshgrid(np.arange(size), np.arange(size), indexing="ij")
    keep = i < j
    src = np.concatenate([c * size + i[keep] for c in range(count)] +
                         [np.arange(count - 1) * size + size - 1])
    dst = np.concatenate([c * size + j[keep] for c in range(count)] +
                         [np.arange(1, count) * size + size - 1])
    return gen.from_edges(count * size, src, dst, np.ones(len(src), np.int32), name="cliques")


def graphs():
    rng = np.random.default_rng(77)
    out = [random_graph(rng, 20000, m, 1, 9, name=f"m{m}")  # rules at 1.5 and 4 edges a vertex
           for m in (1000, 10000, 20000, 29999, 30000, 79999, 80000, 200000)]
    star = gen.from_edges(5001, np.zeros(5000, np.int32) + 5000, np.arange(5000),
                          np.ones(5000, np.int32), name="star-last")
    return out + [path_graph(70000, np.ones(69999)), shuffled_path(70000, 3), cliques(300, 20),
                  star, gen.workload("grid300"), gen.workload("rmat16"),
                  gen.from_edges(70000, [5], [69999], [1], name="one-edge")]


@pytest.mark.parametrize("hg", graphs(), ids=lambda h: h.name)
def test_cc_hooks(hg):
    from paper_1903_01665_amd import gg
    want = oracle.cc(hg.n, hg.row_ptr, hg.col)
    for renumber in (False, True):
        g = gg.Graph.from_host(hg, symmetrize=True, renumber=renumber)
        try:
            for probe in (False, True):
                if probe:
                    g.probe()
                for cap in (0, 3):
                    print(hg.name, renumber, probe, cap, flush=True)
                    o = gg.make_opts(gg.VERTEX, gg.UNIONFIND, max_blocks=cap)
                    np.testing.assert_array_equal(g.cc(opts=o).cpu().numpy(), want)
                    assert g.stats()["iterations"] == 4
                np.testing.assert_array_equal(g.cc().cpu().numpy(), want)
        finally:
            g.free()
