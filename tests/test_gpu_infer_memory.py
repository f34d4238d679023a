"""The allocation calls of the dependence inferences, watched from between the
library and the HIP runtime (tests/native/hip_alloc_shim.c) in a process of
their own."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)  # before whatever loads the runtime
shim.shim_calls.restype = shim.shim_refused.restype = ctypes.c_ulong
shim.shim_limit.argtypes = [ctypes.c_size_t]
import numpy as np, torch
import oracle
from paper_2508_16522_amd import taskgraph as tg
from paper_2508_16522_amd import workloads as wl
from tests.gpu_util import device_requirements, infer_on_device

def watched(fn):
    seen = []
    def call(*a):
        before = shim.shim_calls()
        out = fn(*a)
        seen.append(shim.shim_calls() - before)
        return out
    return call, seen

def same(got, ig):
    row, col = oracle.conflict_dag(ig.N, ig.req_ptr, ig.lo, ig.hi, ig.priv)
    assert np.array_equal(got[0], row) and np.array_equal(got[1], col)
"""


def _run(tmp_path, body):
    so = tmp_path / "hip_alloc_shim.so"
    subprocess.check_call(["gcc", "-O1", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC",
                           os.path.join(ROOT, "tests", "native", "hip_alloc_shim.c"), "-o", str(so), "-ldl"])
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, str(so)], cwd=ROOT, capture_output=True, text=True,
                       timeout=110)
    assert r.returncode == 0 and "done" in r.stdout, r.stdout + r.stderr


def test_the_allocation_free_call_allocates_nothing(gpu, tmp_path):
    # the first calls of a process, then one after an allocating call (which
    # shows that the shim sees the library's calls)
    _run(tmp_path, """
small = wl.halo_graph(16, 64, 9, seed=3, rounds=0)
free, free_calls = watched(tg.tg_infer_dag_noalloc)
alloc, alloc_calls = watched(tg.tg_infer_dag)
same(infer_on_device(small, fn=free), small)
same(infer_on_device(small, fn=free), small)
same(infer_on_device(small, fn=alloc), small)
same(infer_on_device(small, fn=free), small)
assert free_calls == [0, 0, 0], free_calls
assert alloc_calls[0] > 0, "the shim saw nothing"
print("done")
""")
