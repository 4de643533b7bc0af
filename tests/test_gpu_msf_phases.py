"""GPU parity of the minimum spanning forest where its work changes: edge
counts around the lanes' four edges, the 256-edge steps and the switch from
one-step to four-step work items, graphs with and without a light phase, and
weights that leave the light phase nothing to choose (all equal, all largest).
"""
import numpy as np
import pytest

import oracle
from helpers import star
from paper_1903_01665_amd import gen

pytestmark = pytest.mark.gpu
TOP = 2**31 - 1


def uniform(n, m, lo, hi, seed=5):
    rng = np.random.default_rng(seed + n + m)
    return gen.from_edges(n, rng.integers(0, n, m), rng.integers(0, n, m),
                          rng.integers(lo, hi, m, endpoint=True), name=f"u{n}x{m}w{lo}-{hi}")


GRAPHS = [uniform(2, 1, 3, 3), uniform(3, 3, 0, 9), uniform(30, 255, 1, 9),
          uniform(30, 256, 1, 9), uniform(30, 257, 1, 9), uniform(100, 1023, 1, 100),
          uniform(100, 1025, TOP, TOP), uniform(100, 1025, 0, 0), uniform(100, 1025, 0, TOP),
          uniform(1000, 4999, 1, 50), uniform(1000, 5001, 1, 50), uniform(4000, 100000, 1, 3),
          uniform(60000, 50000, 1, 100), uniform(200000, 2097152, 1, 100),
          uniform(200000, 2097153, 1, 100), star(3000, [[7, 7, 2]] * 3000),
          gen.workload("rmat14"), gen.workload("grid63")]


@pytest.mark.parametrize("hg", GRAPHS, ids=lambda h: h.name)
def test_msf_phases(hg):
    from paper_1903_01665_amd import gg
    want = oracle.msf(hg.n, hg.row_ptr, hg.col, hg.w)
    want = np.asarray(want[0] if isinstance(want, tuple) else want).astype(np.uint8)
    for renumber in (False, True):
        g = gg.Graph.from_host(hg, renumber=renumber)
        try:
            for rep in range(2):
                print(hg.name, renumber, rep, flush=True)
                got, weight, edges = g.msf()
                got = got.cpu().numpy()
                np.testing.assert_array_equal(got, want)
                assert edges == int(want.sum())
                assert weight == int(hg.w[want.astype(bool)].astype(np.int64).sum())
            assert g.stats()["rc"] == 0
        finally:
            g.free()
