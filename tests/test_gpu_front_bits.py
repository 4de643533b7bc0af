"""GPU parity of the direction-optimizing BFS around the size from which its
pulled rounds read the frontier as bits: sizes that end inside and at a word
and a tile, hub rows, a symmetric graph, a graph whose frontier grows, shrinks
and grows again, and the blocking, allocation-free and capped forms.
"""
import ctypes

import numpy as np
import pytest

import oracle
from paper_1903_01665_amd import gen

pytestmark = pytest.mark.gpu
N = 1 << 21  # kFrontBitsN


def uniform(n, m, seed, symmetric=False):
    rng = np.random.default_rng(seed)
    src, dst = rng.integers(0, n, m), rng.integers(0, n, m)
    src[:3000] = 7  # a hub row, and a hub's in-list
    dst[3000:6000] = 9
    if symmetric:
        src, dst = np.concatenate([src, dst]), np.concatenate([dst, src])
    return gen.from_edges(n, src, dst, np.ones(len(src), np.int32), name=f"u{n}s{int(symmetric)}",
                          symmetric=symmetric)


def two_waves(n, seed):
    """Two random halves joined by a path: pulled, pushed, pulled again."""
    rng = np.random.default_rng(seed)
    h = n // 2
    a, b = rng.integers(0, h, (2, 4 * h)), rng.integers(h, n - 20, (2, 4 * h))
    chain = np.concatenate([[0], np.arange(n - 20, n), [h]])
    src = np.concatenate([a[0], b[0], chain[:-1]])
    dst = np.concatenate([a[1], b[1], chain[1:]])
    return gen.from_edges(n, src, dst, np.ones(len(src), np.int32), name=f"waves{n}")


@pytest.mark.parametrize("make", [lambda: uniform(N - 1, 9000000, 1), lambda: uniform(N, 9000000, 2),
                                  lambda: uniform(N + 33, 9000000, 3),
                                  lambda: uniform(N + 64, 5000000, 4, True),
                                  lambda: two_waves(N + 4097, 5)])
def test_front_bits(make):
    import torch

    from paper_1903_01665_amd import gg
    hg = make()
    g = gg.Graph.from_host(hg, symmetrize=True)
    try:
        for s in (int(x) for x in gen.pick_sources(hg, 2)):
            want = oracle.bfs(hg.n, hg.row_ptr, hg.col, s)
            for cap in (0, 5):
                o = gg.make_opts(gg.VERTEX, gg.DIROPT, max_blocks=cap)
                for rep in range(2):
                    print(hg.name, s, cap, rep, flush=True)
                    np.testing.assert_array_equal(g.bfs(s, opts=o).cpu().numpy(), want)
            o = gg.make_opts(gg.VERTEX, gg.DIROPT)
            out = torch.full((hg.n,), -1, dtype=torch.int32, device="cuda")
            assert gg.lib().gg_bfs_noalloc(g.handle, s, ctypes.byref(o),
                                           ctypes.c_void_p(out.data_ptr()),
                                           gg._stream_ptr(None)) == 0
            np.testing.assert_array_equal(out.cpu().numpy(), want)
            # the workspace's bitmaps serve the worklist's heavy rows next
            o = gg.make_opts(gg.VERTEX, gg.ASYNC, 3)
            np.testing.assert_array_equal(g.bfs(s, opts=o).cpu().numpy(), want)
    finally:
        g.free()
