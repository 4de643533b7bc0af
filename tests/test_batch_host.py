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
