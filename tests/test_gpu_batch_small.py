"""Batches of instances that one workgroup each could traverse: more than run at
once, so that a workgroup takes several of different sizes in turn; too many
tiny ones; a large one among them, first and last.
"""
import time

import numpy as np
import pytest

import oracle
from helpers import random_graph

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
    run_and_check(inst)


@pytest.mark.parametrize("algo", [0, 1])
def test_a_large_instance_among_tiny_ones(algo):
    graphs, big = tiny(50, 8), large()
    rest = [(algo, g, g.n // 2) for g in graphs * 7]
    for at in (0, 100, len(rest)):
        run_and_check(rest[:at] + [(algo, big, 77)] + rest[at:], 2)


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
