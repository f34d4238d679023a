"""Dependence inferences that fail: what they share with other calls (scratch
arrays, pinned words) is released only once the device has finished with it."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2508_16522_amd import taskgraph as tg
from paper_2508_16522_amd import workloads as wl
from tests.gpu_util import device_requirements, infer_on_device

pytestmark = pytest.mark.gpu


def test_nothing_runs_after_a_refused_call(gpu):
    """440,000 readers of one element: the interval table and the bucket
    entries fit the scratch array, the row counts after them do not.  The
    kernel that fills the entries counts on one address for milliseconds, so a
    call that did not wait for it would return while it still writes the
    array that the next call is given."""
    N = 440_000
    one = np.zeros(N, np.uint64)
    ig = wl.ImplicitGraph(N=N, req_ptr=np.arange(N + 1, dtype=np.uint64), lo=one, hi=one + np.uint64(1),
                          priv=np.full(N, tg.TG_RO, np.uint32), space=1, rounds=0)
    d_ptr, d_reqs = device_requirements(ig)
    row = torch.zeros(N + 1, dtype=torch.int64, device="cuda")
    e = ctypes.c_uint64(7)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    st = tg.load().tg_infer_dag_noalloc(N, ctypes.c_void_p(d_ptr.data_ptr()), ctypes.c_void_p(d_reqs.data_ptr()), N, 1,
                                        ctypes.c_void_p(row.data_ptr()), None, 0, ctypes.byref(e),
                                        ctypes.c_void_p(side.cuda_stream))
    idle = side.query()
    assert st == tg.TG_ENOMEM and b"row counts" in tg.load().tg_last_error()
    assert idle, "the refused call's kernels were still running"
    small = wl.halo_graph(8, 128, 4, seed=2, rounds=1)
    got = infer_on_device(small, fn=tg.tg_infer_dag_noalloc)
    o_row, o_col = oracle.conflict_dag(small.N, small.req_ptr, small.lo, small.hi, small.priv)
    assert np.array_equal(got[0], o_row) and np.array_equal(got[1], o_col)
