"""lfmm_solve_static makes and frees no memory, stream or event, also as the first evaluation of its
context: the calls of a child process to the HIP runtime are counted (tests/native/count_hip_calls.c).
Point sets: a single leaf, a few leaves, and trees whose near field an ordinary solve runs on a stream
of its own beside the far field."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))

CHILD = """
import ctypes, sys
counter = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
counter.counted_calls.restype = ctypes.c_long
sys.path.insert(0, sys.argv[2])
import numpy as np, torch
import paper_1105_3505_amd as lf, workloads as wl
n, side = int(sys.argv[3]), int(sys.argv[4])
rng = np.random.default_rng(n)
xy = torch.from_numpy(np.ascontiguousarray(wl.uniform_box(rng, n, side))).cuda()
f = torch.from_numpy(wl.zero_sum_loads(rng.standard_normal(len(xy)))).cuda()
u = torch.empty(len(xy), dtype=torch.float64, device="cuda")
torch.cuda.synchronize()
before = counter.counted_calls()
ctx = lf.Context(0)
assert counter.counted_calls() > before   # the library's calls are seen
plan = ctx.plan(xy)                # makes the operators; never executed
torch.cuda.synchronize()
before = counter.counted_calls()
ctx.solve_static(xy, f, u)
made = counter.counted_calls() - before
assert made == 0, "%d calls" % made
v = plan.execute(f)
torch.cuda.synchronize()
assert np.array_equal(u.cpu().numpy(), v.cpu().numpy())
plan.close()
ctx.close()
"""


@pytest.mark.parametrize("n,side", [(40, 64), (1000, 256), (16000, 900), (60000, 1000)])
def test_static_solve_makes_nothing(tmp_path, n, side):
    shim = str(tmp_path / "count_hip_calls.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", shim,
                    os.path.join(HERE, "native", "count_hip_calls.c"), "-ldl"], check=True)
    res = subprocess.run([sys.executable, "-c", CHILD, shim, os.path.dirname(HERE), str(n), str(side)],
                         capture_output=True, text=True, timeout=110)
    assert res.returncode == 0, res.stdout + res.stderr
