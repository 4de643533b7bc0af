"""Bytes that bench.py charges kernels for: no more than they must move."""
import bench

N = 1 << 20
NOTHING = {"edges_processed": 0, "vertices_processed": 0, "updates": 0, "pushes": 0}


def test_union_find_rounds_do_not_depend_on_their_launches():
    prof = dict(NOTHING, edges_processed=100, updates=7)
    for launches in (5, 8):
        assert bench.algorithmic_bytes("cc", 0, 5, "round", N, prof, launches) == \
            8 * N + 4 * 100 + 4 * 7
        # init, and a compression at either end
        assert bench.algorithmic_bytes("cc", 0, 5, "aux", N, NOTHING, launches) == 20 * N


def test_launches_that_may_have_returned_at_once_are_not_charged():
    for launches in (1, 2, 40):
        assert bench.algorithmic_bytes("bfs", 0, 4, "aux", N, NOTHING, launches) == 6 * N
