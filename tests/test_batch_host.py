"""What a batch takes, on the host: groups that would be too large together."""
import pytest

from host_hip import run

BATCH = """
def create(shapes):
    inst = (gg.Instance * len(shapes))()
    arrays = {}
    for x, m in zip(inst, shapes):
        if m not in arrays:
            arrays[m] = (np.array([0, m, m], np.int32), np.ones(m, np.int32))
        row, col = arrays[m]
        x.algo, x.n, x.m, x.source = 1, 2, m, 0
        x.row_ptr, x.col = row.ctypes.data, col.ctypes.data
    b = ctypes.c_void_p()
    return L.gg_batch_create(inst, len(shapes), 0, None, ctypes.byref(b))
hip.host_hip_limit(64)  # no graph fits the device: ENOMEM once a group is uploaded
"""


@pytest.mark.parametrize("shapes, rc", [
    ("[131072] * 16383 + [32768] * 4", -2),  # 2^31 edges in two classes
    ("[131072] * 16384", -1),                # 2^31 edges in one class
    ("[131072] * 100 + [32768] * 4", -2)])
def test_groups_of_two_to_the_31_edges(shapes, rc, tmp_path):
    run(BATCH + f"""
got = create({shapes})
print(got)
assert got == {rc}
""", tmp_path)


def test_edge_numbers_of_the_one_launch_stay_in_range(tmp_path):
    """2^31 - 8192 edges are a graph, but the launch counts past its last edge: the
    two classes stay apart.  (Together they are 8 GB of columns, for which the process
    has no room; the small class comes first and finds no device memory.)"""
    run("import resource\nresource.setrlimit(resource.RLIMIT_AS, (6 << 30, 6 << 30))\n" + BATCH +
        """
got = create([131072] * 16383 + [32768] * 3 + [24576])
print(got)
assert got == -2
""", tmp_path)
