"""What a call leaves behind when the runtime refuses something half-way: the library's host code against a stand-in for the HIP
runtime (host_runtime.cpp), in a process of its own."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

VERSIONS = """hip_4.2 { global: hip*; __hip*; };
hip_4.3 { global: hipGraph*; hipStreamBeginCapture; hipStreamEndCapture; } hip_4.2;
"""

CHILD = """
import ctypes as C, sys, types
rt = C.CDLL(sys.argv[1], C.RTLD_GLOBAL)         # stands in for the runtime library the next one asks for
rt.host_runtime_notes.restype = C.c_char_p
sys.modules["torch"] = types.ModuleType("torch")    # (the binding's device memory: the host's, here)
sys.path.insert(0, sys.argv[2])
import numpy as np
from paper_2505_03983_amd import binding as b
L = b.lib()
d, K, n = 8, 6, 16
keep = dict(c_x=np.ones(K, "f4"), c_0=np.ones(K, "f4"), sigma=np.ones(K, "f4"), tau=np.arange(K, 0, -1).astype("i4"),
            abar=np.linspace(1, .1, K + 1).astype("f4"), means=np.zeros((n, d), "f4"), log_w=np.zeros(n, "f4"))
at = {k: v.ctypes.data for k, v in keep.items()}
cfg = b.asd_config()
cfg.sched.K, cfg.L, cfg.chains = K, 4, 2
for k in ("c_x", "c_0", "sigma", "tau"): setattr(cfg.sched, k, at[k])
cfg.den.kind, cfg.den.d, cfg.den.n_tau, cfg.den.C, cfg.den.var = b.ASD_DEN_GMM, d, K + 1, n, 0.25
cfg.den.means, cfg.den.log_w, cfg.den.abar = at["means"], at["log_w"], at["abar"]
ctx = C.c_void_p()
assert L.asd_init(C.byref(cfg), C.byref(ctx)) == 0, L.asd_last_error()
assert L.asd_use_resident(ctx, 0) == 0
traj = np.zeros((2, K + 1, d), "f4")
rt.host_runtime_clear()
rt.host_runtime_fail(sys.argv[3].encode())
s = L.asd_sample(ctx, None, traj.ctypes.data, None, None)
print(s)
print(rt.host_runtime_notes().decode(), end="")
L.asd_destroy(ctx)
"""


@pytest.fixture(scope="module")
def runtime_lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("host_runtime")
    (d / "v.map").write_text(VERSIONS)
    out = str(d / "libamdhip64.so.7")
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-fPIC", "-shared", os.path.join(HERE, "host_runtime.cpp"),
                    "-Wl,-soname,libamdhip64.so.7", "-Wl,--version-script=" + str(d / "v.map"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("failing", ["begin", "instantiate", "launch graph", "query"])
def test_no_round_is_on_the_stream_after_an_error(runtime_lib, failing):
    """Round 0 is queued before the first graph is made: when that fails, asd_sample waits for what it has queued before it
    returns the error, or a later sample could read reports of this one's rounds."""
    r = subprocess.run([sys.executable, "-c", CHILD, runtime_lib, os.path.dirname(HERE), failing], stdout=subprocess.PIPE,
                       stderr=subprocess.PIPE, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    status, *calls = r.stdout.split("\n")[:-1]
    assert int(status) < 0 and "launch" in calls and failing in calls, r.stdout
    assert "synchronize" in calls[calls.index(failing):], r.stdout
