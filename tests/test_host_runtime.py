"""The library's host code against a stand-in for the HIP runtime (host_runtime.cpp), in a process of its own: what a call leaves
behind when the runtime refuses something half-way, and how many graphs a sample makes."""
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

VERSIONS = """hip_4.2 { global: hip*; __hip*; };
hip_4.3 { global: hipGraph*; hipStreamBeginCapture; hipStreamEndCapture; } hip_4.2;
"""

CHILD = """
import ctypes as C, json, sys, types
rt = C.CDLL(sys.argv[1], C.RTLD_GLOBAL)         # stands in for the runtime library the next one asks for
rt.host_runtime_notes.restype = C.c_char_p
sys.modules["torch"] = types.ModuleType("torch")    # (the binding's device memory: the host's, here)
sys.path.insert(0, sys.argv[2])
import numpy as np
from paper_2505_03983_amd import binding as b
L = b.lib()
o = json.loads(sys.argv[3])
d, K, n, W, E = o["d"], o["K"], 16, o.get("width", 8), 8
keep = dict(c_x=np.ones(K, "f4"), c_0=np.ones(K, "f4"), sigma=np.ones(K, "f4"), tau=np.arange(K, 0, -1).astype("i4"),
            abar=np.linspace(1, .1, K + 1).astype("f4"), means=np.zeros((n, d), "f4"), log_w=np.zeros(n, "f4"),
            w_in=np.zeros((W, d + E), "u2"), w_blk=np.zeros((1, W, W), "u2"), w_out=np.zeros((d, W), "u2"),
            temb=np.zeros((K + 1, E), "u2"))
at = {k: v.ctypes.data for k, v in keep.items()}
cfg = b.asd_config()
cfg.sched.K, cfg.L, cfg.chains = K, o["L"], o["chains"]
for k in ("c_x", "c_0", "sigma", "tau"): setattr(cfg.sched, k, at[k])
cfg.den.d, cfg.den.n_tau, cfg.den.C, cfg.den.var = d, K + 1, n, 0.25
cfg.den.kind = b.ASD_DEN_MLP if "width" in o else b.ASD_DEN_GMM
cfg.den.width, cfg.den.n_blocks, cfg.den.linears_per_block, cfg.den.temb_dim, cfg.den.act_terms = W, 1, 1, E, 1
for k in ("means", "log_w", "abar", "w_in", "w_blk", "w_out", "temb"): setattr(cfg.den, k, at[k])
ctx = C.c_void_p()
assert L.asd_init(C.byref(cfg), C.byref(ctx)) == 0, L.asd_last_error()
assert L.asd_use_resident(ctx, 0) == 0
assert L.asd_use_adaptive_window(ctx, int("rounds" in o)) == 0
traj = np.zeros((o["chains"], K + 1, d), "f4")
rt.host_runtime_clear()
if "fail" in o: rt.host_runtime_fail(o["fail"].encode())
if "rounds" in o: rt.host_runtime_rounds((C.c_int * len(o["rounds"]))(*o["rounds"]), len(o["rounds"]))
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


def _sample(runtime_lib, **o):
    r = subprocess.run([sys.executable, "-c", CHILD, runtime_lib, os.path.dirname(HERE), json.dumps(o)], stdout=subprocess.PIPE,
                       stderr=subprocess.PIPE, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    status, *calls = r.stdout.split("\n")[:-1]
    return int(status), calls


@pytest.mark.parametrize("failing", ["begin", "instantiate", "launch graph", "query"])
def test_no_round_is_on_the_stream_after_an_error(runtime_lib, failing):
    """Round 0 is queued before the first graph is made: when that fails, asd_sample waits for what it has queued before it
    returns the error, or a later sample could read reports of this one's rounds."""
    status, calls = _sample(runtime_lib, d=8, K=6, L=4, chains=2, fail=failing)
    assert status < 0 and "launch" in calls and failing in calls, calls
    assert "synchronize" in calls[calls.index(failing):], calls


@pytest.mark.parametrize("chains, forms", [
    (1, 1),       # one chain: the kernel for few rows whatever a round brings
    (90, 3),      # 360 and 720 rows take other tiles than 1440, which take those of all 2070
])
def test_rounds_launched_alike_share_a_graph(runtime_lib, chains, forms):
    """Windows by the controller, a network 1536 wide: rounds that bring from 4 rows a chain to all 23 are launched for as many,
    and a graph is made for every choice of tiles, not for every count."""
    rows = [chains * n for n in (23, 3, 7, 15, 22, 23, 3, 7, 15, 22)] + [0]
    status, calls = _sample(runtime_lib, d=768, K=30, L=24, chains=chains, width=1536, rounds=rows)
    assert status == 0 and calls.count("launch graph") == len(rows) + 1
    assert calls.count("instantiate") == forms
