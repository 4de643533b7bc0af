"""Which calls run as one workgroup, and what that launch counts."""
import numpy as np
import pytest

import oracle
from helpers import random_graph
from paper_1903_01665_amd import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [0, 1, 1000, 4095, 4096, 4097, 20001])
def test_cc_counts_each_edge_once(m):
    from paper_1903_01665_amd import gg
    hg = random_graph(np.random.default_rng(m), 700, m)
    g = gg.Graph.from_host(hg)
    try:
        np.testing.assert_array_equal(g.cc().cpu().numpy(),
                                      oracle.cc(hg.n, hg.row_ptr, hg.col))
        assert g.stats()["edges_processed"] == m
    finally:
        g.free()


@pytest.mark.parametrize("order", ["up", "down", "shuffled"])
def test_cc_of_a_chain(order):
    """The links of a path in order make one chain; no lane walks all of it
    (32,767 dependent reads of LDS take more than a millisecond)."""
    import time

    import torch

    from paper_1903_01665_amd import gg
    p = np.arange(32768, dtype=np.int32)
    p = {"up": p, "down": p[::-1], "shuffled": np.random.default_rng(4).permutation(p)}[order]
    hg = gen.from_edges(len(p), p[:-1], p[1:], np.ones(len(p) - 1, np.int32), name=order)
    for renumber in (None, True):
        g = gg.Graph.from_host(hg, renumber=renumber)
        try:
            times = []
            for _ in range(6):
                t = time.perf_counter()
                c = g.cc()
                torch.cuda.synchronize()
                times.append(1e3 * (time.perf_counter() - t))
                assert int(c.max()) == 0
            print(order, renumber, times, flush=True)
            assert min(times) < 0.7
        finally:
            g.free()
