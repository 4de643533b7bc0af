"""Run a script against libgg.so over the host stand-in of HIP (host_hip.c), in a
process of its own: host paths that need a device's failures or sizes."""
import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys, time
import numpy as np
hip = ctypes.CDLL({fake!r}, mode=ctypes.RTLD_GLOBAL)
hip.host_hip_limit.argtypes = [ctypes.c_size_t]
hip.host_hip_launches.restype = ctypes.c_long
from paper_1903_01665_amd import gg
L = ctypes.CDLL(gg.LIB_PATH)
P = lambda a: ctypes.c_void_p(a.ctypes.data)
def upload(n, src, dst, flags=0):
    order = np.argsort(src, kind="stable")
    row = np.zeros(n + 1, np.int32)
    row[1:] = np.cumsum(np.bincount(src, minlength=n))
    col = np.asarray(dst, np.int32)[order]
    w = np.ones(len(col), np.int32)
    g = ctypes.c_void_p()
    assert L.gg_graph_upload(n, ctypes.c_int64(len(col)), P(row), P(col), P(w), flags, None,
                             ctypes.byref(g)) == 0
    return g
"""


def run(script, tmp_path, timeout=60):
    fake = os.path.join(str(tmp_path), "host_hip.so")
    subprocess.run(["gcc", "-std=gnu11", "-O1", "-shared", "-fPIC",
                    os.path.join(HERE, "host_hip.c"), "-o", fake], check=True)
    code = PRELUDE.format(fake=fake) + textwrap.dedent(script)
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, text=True, timeout=timeout)
    assert r.returncode == 0, r.stdout
    return r.stdout
