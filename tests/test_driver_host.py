"""The blocking driver on the host: what a call returns, and when, if the device
never reports a round."""
import pytest

from host_hip import run

CALLS = """
n = 50000
g = upload(n, np.arange(n - 1), np.arange(1, n), gg.SYMMETRIZE)
out = np.zeros(n, np.int32)
def call(algo, ms, sched=gg.ASYNC):
    o = gg.Opts(mode=gg.VERTEX, sched=sched, mapping=gg.MAP_BALANCED, time_limit_ms=ms)
    t = time.perf_counter()
    if algo == "cc":
        rc = L.gg_cc_ex(g, None, ctypes.byref(o), P(out), None)
    else:
        rc = getattr(L, "gg_%s_ex" % algo)(g, None, 0, ctypes.byref(o), P(out), None)
    return rc, time.perf_counter() - t
"""


@pytest.mark.parametrize("algo, sched", [("sssp", "ASYNC"), ("bfs", "SYNC"), ("cc", "UNIONFIND")])
def test_a_failed_kernel_is_reported_at_once(algo, sched, tmp_path):
    """hipErrorLaunchFailure, with 20 s left of the call's time."""
    run(CALLS + f"""
hip.host_hip_answer(719)
rc, t = call({algo!r}, 20000, gg.{sched})
print(rc, t)
assert rc == -3 and t < 5
assert L.gg_graph_error(g) == -3
""", tmp_path)


def test_a_round_that_takes_long_is_waited_for(tmp_path):
    """The time limit ends the call, not before it is over; the rounds enqueued by
    then are those that go ahead of the device, and the core is not kept busy."""
    run(CALLS + """
before = hip.host_hip_launches()
cpu = time.thread_time()
rc, t = call("bfs", 400)
cpu = time.thread_time() - cpu
print(rc, t, cpu, hip.host_hip_launches() - before)
assert rc == -6 and 0.4 <= t < 5
assert hip.host_hip_launches() - before < 20
assert cpu < 0.2
assert L.gg_graph_error(g) == 0
""", tmp_path)
