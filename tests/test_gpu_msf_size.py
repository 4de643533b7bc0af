"""The minimum spanning forest around the edge count from which it has a light
phase: both sides of it, and weights that leave that phase nothing to choose.
"""
import numpy as np
import pytest

import oracle
from helpers import star
from paper_1903_01665_amd import gen

pytestmark = pytest.mark.gpu
TOP, LEAST = 2**31 - 1, 1 << 18  # kLightLeast


def uniform(n, m, lo, hi):
    rng = np.random.default_rng(n + m + hi)
    return gen.from_edges(n, rng.integers(0, n, m), rng.integers(0, n, m),
                          rng.integers(lo, hi, m, endpoint=True), name=f"u{n}x{m}w{lo}-{hi}")


def bundles(leaves, parallel):
    """A star with `parallel` edges to each leaf, of as many weights."""
    return star(leaves, [[1 + (i * 5 + k * 7) % 97 for k in range(parallel)]
                         for i in range(leaves)])


@pytest.mark.parametrize("hg", [
    uniform(100, LEAST - 1, 0, TOP), uniform(100, LEAST, 0, TOP), uniform(100, LEAST + 1, 0, TOP),
    uniform(30000, LEAST, 7, 7), uniform(30000, LEAST + 3, TOP, TOP), uniform(30000, LEAST, 0, 1),
    uniform(52428, LEAST, 1, 100), uniform(52429, LEAST, 1, 100), bundles(32768, 8),
    uniform(30000, LEAST + 257, 1, 100)], ids=lambda h: f"{h.name}{h.n}")
def test_around_the_light_phase(hg):
    from paper_1903_01665_amd import gg
    want = oracle.msf(hg.n, hg.row_ptr, hg.col, hg.w)
    want = np.asarray(want[0] if isinstance(want, tuple) else want).astype(np.uint8)
    for renumber in (False, True):
        g = gg.Graph.from_host(hg, renumber=renumber)
        try:
            print(hg.name, hg.n, renumber, flush=True)
            for _ in range(2):
                got, weight, edges = g.msf()
                np.testing.assert_array_equal(got.cpu().numpy(), want)
                assert edges == int(want.sum())
                assert weight == int(hg.w[want.astype(bool)].astype(np.int64).sum())
        finally:
            g.free()


@pytest.mark.parametrize("leaves, phases", [(100, 1), (32767, 1), (32768, 2)])
def test_rounds(leaves, phases):
    """One round joins a star and the next finds it joined; a light phase before it
    has two rounds of its own."""
    from paper_1903_01665_amd import gg
    g = gg.Graph.from_host(bundles(leaves, 8))
    try:
        g.msf()
        assert (g.stats()["iterations"] <= 2) == (phases == 1)
    finally:
        g.free()
