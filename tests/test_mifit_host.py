"""Host side of the gradient search, on the CPU: what a call asks of the HIP
runtime, recorded by a stand-in for it (native/gs_launch_shim.cpp)."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(ROOT, "paper_2209_10411_amd", "libmidelbm.so")

CALLS = """
import ctypes as C
import sys
import numpy as np
L = C.CDLL(sys.argv[1])
vp = C.c_void_p
L.mi_gs.argtypes = [vp, vp, vp, vp, C.c_int32, C.c_int32, C.c_int32, C.c_double, vp, vp, vp]
p = lambda a: a.ctypes.data_as(vp)
for m in (64, 2900, 3072, 3073, 6144, 5):
    ho, po = np.array([0, m], np.int64), np.array([0, 1], np.int64)
    H, pl, M, loss = np.zeros((m, 3)), np.zeros((1, 4)), np.zeros((1, 8, 4)), np.zeros(3)
    rc = L.mi_gs(p(H), p(ho), p(pl), p(po), 1, 8, 2, 1e-5, p(M), p(loss), None)
    print("call", m, rc, flush=True)
"""


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    d = tmp_path_factory.mktemp("shim")
    so = str(d / "shim.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "native", "gs_launch_shim.cpp")],
                   check=True)
    r = subprocess.run([sys.executable, "-c", CALLS, LIB], env={**os.environ, "LD_PRELOAD": so}, capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    return [line.split() for line in r.stdout.splitlines()]


def test_gradient_search_limits_do_not_depend_on_the_call(record):
    """A kernel's dynamic LDS limit belongs to the kernel, for every thread of
    the process: all calls that set it set the same value, which holds every
    launch of that kernel."""
    assert [r[1:] for r in record if r[0] == "call"] == [[str(m), "0"] for m in (64, 2900, 3072, 3073, 6144, 5)]
    limits, launches = {}, {}
    for r in record:
        if r[0] == "limit":
            limits.setdefault(r[1], set()).add(int(r[3]))
        elif r[0] == "launch":
            launches.setdefault(r[1], []).append(int(r[4]))
    assert launches and sum(map(len, launches.values())) == 6
    for k, v in limits.items():
        assert len(v) == 1, (k, v)
        assert max(launches.get(k, [0])) <= min(v)
