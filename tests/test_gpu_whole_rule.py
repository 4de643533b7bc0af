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


def grid(w, h):
    return gen.grid(w, h, 0, 8, 1, 1000, stream=w)


def star(n):
    return gen.from_edges(n, np.zeros(n - 1, np.int32), np.arange(1, n), np.ones(n - 1, np.int32),
                          name=f"star{n}")


def uniform(n, m):
    return random_graph(np.random.default_rng(n + m), n, m, 1, 100)


# (graph, probed, which of SSSP, BFS and CC run as one workgroup)
RULE = [(uniform(32768, 32768), False, "sbc"), (uniform(32769, 32768), False, ""),
        (uniform(5000, 32768), True, "sbc"), (uniform(5000, 32769), True, "sc"),
        (uniform(5000, 65536), False, "sc"), (uniform(5000, 65537), False, ""),
        (grid(39, 40), True, "sbc"), (grid(40, 40), True, "sc"), (grid(55, 56), True, "sc"),
        (grid(56, 56), True, "c"), (grid(4, 200), True, "sbc"), (grid(4, 300), True, "c"),
        (grid(64, 64), False, "sbc"),
        (grid(64, 64), True, "c"), (grid(109, 110), False, "sc"), (grid(110, 110), False, "c"),
        (star(20480), False, "sbc"), (star(20481), True, "c")]


@pytest.mark.parametrize("hg, probed, whole", RULE, ids=lambda x: getattr(x, "name", str(x)))
def test_which_calls_run_as_one_workgroup(hg, probed, whole):
    from paper_1903_01665_amd import gg
    g = gg.Graph.from_host(hg)
    try:
        if probed:
            g.probe()
        s = hg.n // 2
        want = {"s": oracle.sssp(hg.n, hg.row_ptr, hg.col, hg.w, s),
                "b": oracle.bfs(hg.n, hg.row_ptr, hg.col, s),
                "c": oracle.cc(hg.n, hg.row_ptr, hg.col)}
        calls = {"s": lambda **k: g.sssp(s, **k), "b": lambda **k: g.bfs(s, **k), "c": g.cc}
        for k, call in calls.items():
            np.testing.assert_array_equal(call().cpu().numpy(), want[k])
            assert g.stats()["block_threads"] == (1024 if k in whole else 256), k
            for o in (dict(mode=gg.EDGE, sched=gg.SYNC), dict(mapping=gg.MAP_BALANCED),
                      dict(time_limit_ms=60000)):
                np.testing.assert_array_equal(call(opts=gg.make_opts(**o)).cpu().numpy(), want[k])
                assert g.stats()["block_threads"] == 256, (k, o)
    finally:
        g.free()
