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
