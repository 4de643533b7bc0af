"""The direction-optimizing BFS makes a frontier into bits in its first rounds
only: levels that pull before, at and after the last of them, on graphs kept in
the caller's order (a hub alone would have them renumbered), with rows and
in-lists long enough to share the bitmap with the bits.
"""
import numpy as np
import pytest

import oracle
from paper_1903_01665_amd import gen

pytestmark = pytest.mark.gpu
N, ROUNDS = 1 << 21, 32  # kFrontBitsN, kFrontBitsRounds


def lollipop(tail, n, symmetric):
    """A path of `tail` edges into a uniform graph, whose wide levels pull."""
    rng = np.random.default_rng(tail)
    src = np.r_[np.arange(tail), rng.integers(tail, n, 3 * n)]
    dst = np.r_[np.arange(1, tail + 1), rng.integers(tail, n, 3 * n)]
    src[-5000:] = tail + 5  # a long row
    dst[-9000:-6000] = tail + 9  # a long in-list
    if symmetric:
        src, dst = np.r_[src, dst], np.r_[dst, src]
    return gen.from_edges(n, src, dst, np.ones(len(src), np.int32), name=f"tail{tail}",
                          symmetric=symmetric)


@pytest.mark.parametrize("tail, n, symmetric", [
    (0, N, False), (0, N + 31, True), (ROUNDS - 8, N, False), (ROUNDS - 5, N + 64, False),
    (ROUNDS - 4, N + 1, False), (ROUNDS - 3, N, True), (ROUNDS, N, False), (70, N, False)])
def test_levels_around_the_last_round_with_bits(tail, n, symmetric):
    from paper_1903_01665_amd import gg
    hg = lollipop(tail, n, symmetric)
    g = gg.Graph.from_host(hg, symmetrize=True, renumber=False)
    try:
        assert not g.renumbered()
        s = tail + 5 if tail == 0 else 0
        want = oracle.bfs(hg.n, hg.row_ptr, hg.col, s)
        assert np.bincount(want[want < hg.n]).max() * 16 > n  # some level pulls
        for flags in (0, gg.OPT_PROFILE):
            o = gg.make_opts(gg.VERTEX, gg.DIROPT, flags=flags)
            np.testing.assert_array_equal(g.bfs(s, opts=o).cpu().numpy(), want)
        assert g.profile()["aux"]["launches"] <= ROUNDS
        # the workspace's bitmaps serve the worklist's heavy rows next
        np.testing.assert_array_equal(
            g.bfs(s, opts=gg.make_opts(gg.VERTEX, gg.ASYNC, gg.MAP_BALANCED)).cpu().numpy(), want)
    finally:
        g.free()
