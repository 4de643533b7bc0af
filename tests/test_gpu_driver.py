"""The blocking driver's waits: behind other work of its stream for longer than it
spins, and past a time limit, whatever the schedule; the workspace serves the next
call as before.
"""
import numpy as np
import pytest

import oracle
from helpers import path_graph, random_graph

pytestmark = pytest.mark.gpu
ETIMEOUT = -6


@pytest.mark.parametrize("renumber", [False, True])
def test_behind_other_work(renumber):
    import torch

    from paper_1903_01665_amd import gg
    hg = random_graph(np.random.default_rng(1), 60000, 400000, 1, 100)
    g = gg.Graph.from_host(hg, symmetrize=True, renumber=renumber)
    a = torch.ones(8192, 8192, device="cuda", dtype=torch.bfloat16)
    try:
        want = (oracle.sssp(hg.n, hg.row_ptr, hg.col, hg.w, 5),
                oracle.bfs(hg.n, hg.row_ptr, hg.col, 5), oracle.cc(hg.n, hg.row_ptr, hg.col))
        for stream in (torch.cuda.current_stream(), torch.cuda.Stream()):
            with torch.cuda.stream(stream):
                for call, w in zip((lambda: g.sssp(5), lambda: g.bfs(5), lambda: g.cc()), want):
                    for _ in range(30):  # about 1 ms each
                        b = a @ a
                    print(renumber, stream, flush=True)
                    np.testing.assert_array_equal(call().cpu().numpy(), w)
        del b
    finally:
        g.free()


@pytest.mark.parametrize("mode, sched", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_time_limit(mode, sched):
    from paper_1903_01665_amd import gg
    hg = path_graph(60000, np.ones(59999))
    g = gg.Graph.from_host(hg, symmetrize=True)
    try:
        for renumber in (False, True):
            with pytest.raises(gg.GGError) as e:
                g.bfs(0, opts=gg.make_opts(mode, sched, time_limit_ms=3))
            assert e.value.code == ETIMEOUT
            with pytest.raises(gg.GGError) as e:  # gg_last_stats returns the run's status
                gg._check(gg.lib().gg_last_stats(g.handle, None, gg.ctypes.byref(gg.Stats())), "")
            assert e.value.code == ETIMEOUT
            np.testing.assert_array_equal(g.bfs(59000).cpu().numpy(),
                                          oracle.bfs(hg.n, hg.row_ptr, hg.col, 59000))
            g.free()
            g = gg.Graph.from_host(hg, symmetrize=True, renumber=True)
    finally:
        g.free()
