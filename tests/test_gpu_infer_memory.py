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


@pytest.mark.parametrize("limit", [1 << 26, 20 << 20])
def test_entries_beyond_the_device_memory(gpu, tmp_path, limit):
    """800,000 writers of one element each, eight to an element: 38 MB of
    entries by their number, 115 MB by the bound on it.  Where the device has
    room for the former, or only for the smaller tables of the other pipeline
    (no allocation above `limit` succeeds), the call still works."""
    _run(tmp_path, f"""
N, S = 800_000, 100_000
k = np.arange(N, dtype=np.uint64)
lo = k % np.uint64(S)
ig = wl.ImplicitGraph(N=N, req_ptr=np.arange(N + 1, dtype=np.uint64), lo=lo, hi=lo + np.uint64(1),
                      priv=np.full(N, tg.TG_RW, np.uint32), space=S, rounds=0)
later = (N - 1 - np.arange(N)) // S
def limited(*a):
    shim.shim_limit({limit})
    try:
        return tg.tg_infer_dag(*a)
    finally:
        shim.shim_limit(1 << 60)
row, col = infer_on_device(ig, col_cap=int(later.sum()), fn=limited)
ref = np.zeros(N + 1, np.uint64)
ref[1:] = np.cumsum(later)
assert np.array_equal(row, ref)
assert np.array_equal(col, np.repeat(np.arange(N), later) + S * (1 + np.arange(col.size) - np.repeat(ref[:-1].astype(np.int64), later)))
if {limit} < 30_000_000: assert shim.shim_refused() > 0
print("done")
""")
