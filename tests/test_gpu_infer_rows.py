"""The rows of the device inference where their kernel changes behaviour: rows
of more than one bitmap window (programs of more than 65,536 tasks), tasks of
more than 64 entries, lists longer than a wavefront, buckets of one or many
intervals, intervals of one task sharing a bucket, and requirement lists whose
entries do not fit the scratch array of the allocation-free entry point.  The
reference is the oracle's brute force, or a closed form where the program is
too large for it."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_16522_amd import taskgraph as tg
from paper_2508_16522_amd import workloads as wl
from tests.gpu_util import infer_on_device

pytestmark = pytest.mark.gpu


def _program(rows, space):
    """ImplicitGraph of a list of tasks, each a list of (lo, hi, priv)."""
    ptr = np.zeros(len(rows) + 1, np.uint64)
    ptr[1:] = np.cumsum([len(r) for r in rows])
    flat = np.array([q for r in rows for q in r], np.uint64).reshape(-1, 3)
    return wl.ImplicitGraph(N=len(rows), req_ptr=ptr, lo=flat[:, 0].copy(), hi=flat[:, 1].copy(),
                            priv=flat[:, 2].astype(np.uint32), space=space, rounds=0)


def _check(ig):
    row, col = oracle.conflict_dag(ig.N, ig.req_ptr, ig.lo, ig.hi, ig.priv)
    for fn in (tg.tg_infer_dag, tg.tg_infer_dag_noalloc):
        got = infer_on_device(ig, fn=fn)
        assert np.array_equal(got[0], row), fn.__name__
        assert np.array_equal(got[1], col), fn.__name__


@pytest.mark.parametrize("intervals", [1, 2, 5, 63, 64, 65, 150])
def test_entries_per_task(gpu, intervals):
    # single elements every 7, each its own entry; and one interval over many
    # buckets beside them (the median length stays one element)
    rng = np.random.default_rng(intervals)
    rows = []
    for _ in range(70):
        at = rng.choice(400, size=intervals, replace=False) * 7
        rows.append([(a, a + 1, 1 + int(rng.integers(0, 2))) for a in np.sort(at)])
    rows.append([(0, 2800, 2)])
    rows.append([(100, 1900, 1), (1900, 1901, 2)])
    _check(_program(rows, 2801))


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 129, 300])
@pytest.mark.parametrize("writers", ["all", "none", "some"])
def test_one_bucket(gpu, n, writers):
    # every task in one bucket, each with two intervals there (read-only ones
    # before and after a read-write one)
    rng = np.random.default_rng(n)
    rows = []
    for i in range(n):
        w = 2 if writers == "all" or (writers == "some" and i % 3 == 0) else 1
        a, b = int(rng.integers(0, 30)), int(rng.integers(60, 90))
        rows.append([(a, a + int(rng.integers(0, 30)), 1), (60 - i % 2, 60, w), (b, b + 10, 1)])
    _check(_program(rows, 128))


@pytest.mark.parametrize("seed", range(6))
def test_random_lengths(gpu, seed):
    # interval lengths over several orders of magnitude, clustered starts
    rng = np.random.default_rng(100 + seed)
    space = [1000, 1 << 20, 1 << 36][seed % 3]
    rows = []
    for _ in range(257):
        lo = int(rng.integers(0, 40)) * (space // 41)
        ln = int(min(space - lo, np.exp(rng.uniform(0, np.log(space / 20)))))
        rows.append([(lo, lo + ln, 1 + int(rng.random() < 0.4))])
    _check(_program(rows, space))


def test_wide_buckets(gpu):
    # intervals longer than 2^31 elements: a bucket's offsets no longer fit 32
    # bits, so the index tables run
    rows = [[(i << 33, (i << 33) + (5 << 32), 1 + i % 2)] for i in range(6)]
    _check(_program(rows, 1 << 36))


@pytest.mark.parametrize("N", [65536, 65537, 65538, 131073, 200000])
def test_many_tasks(gpu, N):
    """Tasks 0 and 1 write elements everybody else reads in turn (element 0 by
    even tasks, 1 by odd ones), the last two tasks write them again: rows that
    cross every window, rows with one successor in the last window, and empty
    stretches in between (each task also writes an element of its own)."""
    k = np.arange(N, dtype=np.int64)
    last = k >= N - 2
    shared = np.where(last, k - (N - 2), k % 2)
    lo = np.stack([shared, 2 + k], 1).reshape(-1).astype(np.uint64)
    priv = np.stack([np.where((k < 2) | last, 2, 1), np.full(N, 2)], 1).reshape(-1).astype(np.uint32)
    ig = wl.ImplicitGraph(N=N, req_ptr=np.arange(N + 1, dtype=np.uint64) * np.uint64(2), lo=lo, hi=lo + np.uint64(1),
                          priv=priv, space=N + 2, rounds=0)
    ends = {p: N - 2 + p for p in (0, 1)}  # the task that writes element p again
    want = [np.concatenate([k[(k > 1) & (k % 2 == p) & ~last], [ends[p]]]) for p in (0, 1)]
    counts = np.where(last, 0, 1)
    counts[:2] = [w.size for w in want]
    row_ref = np.zeros(N + 1, np.uint64)
    row_ref[1:] = np.cumsum(counts)
    row, col = infer_on_device(ig, col_cap=int(row_ref[-1]))
    assert np.array_equal(row, row_ref)
    assert np.array_equal(col[:want[0].size], want[0]) and np.array_equal(col[want[0].size:row[2]], want[1])
    rest = np.arange(2, N - 2)
    assert np.array_equal(col[int(row[2]):], N - 2 + rest % 2)


def test_near_the_scratch_limit(gpu):
    """380,000 requirements: within what the allocation-free entry point takes
    (its older tables), past what the sorted entries would.  Task k has two
    intervals in 8192 slots of 16 elements, every thousandth task writes one."""
    N, slots = 190_000, 8192
    k = np.arange(N, dtype=np.int64)
    lo = 16 * np.stack([k % slots, (k * 7 + 1) % slots], 1)
    priv = np.ones((N, 2), np.uint32)
    priv[::1000, 0] = 2
    same = lo[:, 0] == lo[:, 1]
    lo[same, 1] = 16 * ((k[same] + 1) % slots)
    ig = wl.ImplicitGraph(N=N, req_ptr=np.arange(N + 1, dtype=np.uint64) * np.uint64(2), lo=lo.reshape(-1).astype(np.uint64),
                          hi=(lo + 16).reshape(-1).astype(np.uint64), priv=priv.reshape(-1), space=16 * slots, rounds=0)
    a = infer_on_device(ig, col_cap=1 << 20)
    b = infer_on_device(ig, col_cap=1 << 20, fn=tg.tg_infer_dag_noalloc)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and a[1].size > 5000
    for j in [0, 1, 999, 1000, 1001, 8192, 100_000, 189_000, N - 1]:
        want = oracle.conflict_row(ig.N, ig.req_ptr, ig.lo, ig.hi, ig.priv, j)
        assert np.array_equal(a[1][int(a[0][j]):int(a[0][j + 1])], want), f"row {j}"


def test_capacity_below_the_edge_count(gpu):
    # nothing is written past or into a column array that is too small
    ig = wl.halo_graph(16, 64, 9, seed=3, rounds=0)
    row, col = oracle.conflict_dag(ig.N, ig.req_ptr, ig.lo, ig.hi, ig.priv)
    from tests.gpu_util import device_requirements
    import ctypes
    d_ptr, d_reqs = device_requirements(ig)
    d_row = torch.zeros(ig.N + 1, dtype=torch.int64, device="cuda")
    d_col = torch.full((col.size,), -7, dtype=torch.int32, device="cuda")
    e = ctypes.c_uint64()
    st = tg.load().tg_infer_dag(ig.N, ctypes.c_void_p(d_ptr.data_ptr()), ctypes.c_void_p(d_reqs.data_ptr()),
                                int(ig.lo.size), ig.space, ctypes.c_void_p(d_row.data_ptr()),
                                ctypes.c_void_p(d_col.data_ptr()), col.size - 1, ctypes.byref(e), None)
    assert st == tg.TG_ENOMEM and e.value == col.size
    assert (d_col == -7).all()


@pytest.mark.parametrize("readers", [1, 2, 5])
def test_whole_array_readers(gpu, readers):
    """A halo program whose sweeps each end with tasks that read the whole array
    (one of them also writes a word of its own): most declared elements are theirs,
    and they have an entry in every bucket."""
    P, S, sweeps = 48, 700, 12
    rows = []
    for k in range(sweeps):
        for p in range(P):
            row = [(p * S, p * S + S, 2)]
            if p:
                row.append((p * S - 5 - k, p * S, 1))
            if p + 1 < P:
                row.append((p * S + S, p * S + S + 17, 1))
            rows.append(row)
        rows += [[(0, P * S, 1)] + ([(P * S + k, P * S + k + 1, 2)] if r == 0 else []) for r in range(readers)]
    _check(_program(rows, P * S + sweeps))
