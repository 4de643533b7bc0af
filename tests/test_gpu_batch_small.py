"""Batches of instances that one workgroup each could traverse: more than run at
once, so that a workgroup takes several of different sizes in turn; too many
tiny ones; a large one among them, first and last; a deep one.
"""
import time

import numpy as np
import pytest

import oracle
from helpers import path_graph, random_graph
from paper_1903_01665_amd import gen

pytestmark = pytest.mark.gpu


def tiny(count, seed):
    """Graphs of 1 to 130 vertices and 0 to 900 edges."""
    rng = np.random.default_rng(seed)
    return [random_graph(rng, int(rng.integers(1, 131)), int(rng.integers(0, 900)), 0, 50)
            for _ in range(count)]


def large():
    return random_graph(np.random.default_rng(3), 20000, 131072, 1, 100)


def run_and_check(inst, reps=3):
    import torch

    from paper_1903_01665_amd import gg
    known = {}
    b = gg.Batch(inst)
    try:
        out = torch.empty(b.total_n, dtype=torch.int32, device="cuda")
        for _ in range(reps):
            out.fill_(-7)
            b.run(out)
            got = out.cpu().numpy()
            for o, (a, h, s) in zip(b.offsets(), inst):
                key = (a, id(h), s)
                if key not in known:
                    known[key] = oracle.sssp(h.n, h.row_ptr, h.col, h.w, s) if a == 0 else \
                        oracle.bfs(h.n, h.row_ptr, h.col, s)
                np.testing.assert_array_equal(got[o:o + h.n], known[key])
        return [b.group(i) for i in range(b.info()["groups"])]
    finally:
        b.free()


@pytest.mark.parametrize("algo", [0, 1])
@pytest.mark.parametrize("count", [255, 257, 700, 5000])
def test_many_tiny_instances(algo, count):
    graphs = tiny(90, count)
    inst = [(algo, graphs[i % 90], (i * 7) % graphs[i % 90].n) for i in range(count)]
    print(algo, count, flush=True)
    groups = run_and_check(inst)
    if algo == 0:  # one launch up to 512 + 2.5 edges an instance
        assert (len(groups) == 1) == (count < 1500)


@pytest.mark.parametrize("algo", [0, 1])
def test_a_large_instance_among_tiny_ones(algo):
    graphs, big = tiny(50, 8), large()
    rest = [(algo, g, g.n // 2) for g in graphs * 7]
    for at in (0, 100, len(rest)):
        run_and_check(rest[:at] + [(algo, big, 77)] + rest[at:], 2)


@pytest.mark.parametrize("algo", [0, 1])
def test_sparse_instances_above_65536_edges_run_in_rounds(algo):
    """... as they may be deep; the others, small or with more edges a vertex,
    are one launch beside them."""
    grid = gen.grid(160, 160, 0, 8, 1, 1000, stream=5)  # 101,760 edges, no long row
    graphs = [random_graph(np.random.default_rng(1), 5000, 30000, 1, 9),
              path_graph(3000, np.ones(2999)), large()]
    groups = run_and_check([(algo, g, 5) for g in graphs] + [(algo, grid, 0)])
    assert sorted(g["instances"] for g in groups) == [1, 3]
    # its rounds are launches: as many as its depth asks for
    assert [g["captured_rounds"] > 10 for g in groups if g["instances"] == 1] == [True]


@pytest.mark.parametrize("algo, few, many", [(0, 4, 8), (1, 16, 24)])
def test_a_few_large_instances_stay_out_of_the_launch(algo, few, many):
    """Their rounds are faster than the launch that waits for one of them."""
    hub = gen.rmat(13, 1 << 17, stream=6)
    small = [(algo, g, 0) for g in tiny(20, 5)]
    for count in (few, many):
        groups = run_and_check(small + [(algo, hub, i) for i in range(count)], 2)
        assert sorted(g["instances"] for g in groups) == \
            ([20 + many] if count == many else sorted([20, few]))


@pytest.mark.parametrize("algo", [0, 1])
def test_tiny_instances_do_not_cost_a_workgroup_each(algo):
    """Sixteen times the instances, of 64 edges, in less than three times the time
    (a workgroup each: five times)."""
    import torch

    from paper_1903_01665_amd import gg
    g = random_graph(np.random.default_rng(2), 16, 64, 1, 9)
    best = []
    for count in (250, 4000):
        b = gg.Batch([(algo, g, 0)] * count)
        try:
            out = torch.empty(b.total_n, dtype=torch.int32, device="cuda")
            times = []
            for _ in range(8):
                t = time.perf_counter()
                b.run(out)
                torch.cuda.synchronize()
                times.append(time.perf_counter() - t)
            best.append(min(times))
        finally:
            b.free()
    print(algo, best, flush=True)
    assert best[1] < 3 * best[0]
