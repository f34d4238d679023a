"""Performance cases of the task-DAG executor: the calls a program makes of
this library, each through its public entry points, over the sizes its
configurations, tests and benchmark use.

A case is a dict of plain values:

  kind "graph"   one explicit graph (pattern, W x T tasks, n-word payloads, R
                 mix rounds), executed and its results read;
  kind "steps"   several Task Bench patterns of one size in one batched launch
                 (the benchmark's step);
  kind "batch"   independent uneven graphs in one launch;
  kind "halo"    an implicit halo program (P subregions of S elements, `iters`
                 sweeps), executed and its array read;
  kind "infer"   dependence inference of a halo program's requirements held in
                 device memory, its sweeps starting at a seeded subregion;
  kind "regions" the same for tasks over uneven subregions, each writing part
                 of one and reading parts of others;
  kind "serve"   a burst of requests through the continuous-batching server.

All results are integers and must agree exactly.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2508_16522_amd import taskgraph as tg
from paper_2508_16522_amd import workloads as wl

# Launch shapes by name: the library's defaults, and the shapes the benchmark
# and the autotuner settle on for these workloads.
SHAPES = {
    "default": None,
    # a column of a Task Bench graph kept on one wavefront
    "column": dict(mapping=tg.TG_MAP_WAVE, schedule=tg.TG_SCHED_COLUMN),
    "queue": dict(mapping=tg.TG_MAP_WAVE, workers=2048, dispatch=tg.TG_DISPATCH_QUEUE, tile=1),
    "workgroup": dict(mapping=tg.TG_MAP_WORKGROUP, wg_waves=4),
    # tasks of very different costs
    "balanced": dict(mapping=tg.TG_MAP_WAVE, workers=4096, schedule=tg.TG_SCHED_BALANCED, idle_sleep=32),
    # few, large tasks: several workgroups per task
    "gang": dict(mapping=tg.TG_MAP_GANG, workers=96, wg_waves=8, gang=8, schedule=tg.TG_SCHED_COLUMN),
}

ROUND_OPS = 8   # three shifts, three xors, a multiply and an add
REQ_BYTES = 24  # sizeof(tg_region_req)


def listed():
    return [
        # the smallest graph of the tests and the smoke check: launches, 16
        # dependent levels and the read-back of 128 digests
        dict(name="stencil_8x16", kind="graph", pattern="stencil", W=8, T=16, n=64, rounds=16, shape="default"),
        # an ordinary graph of ragged width (the butterfly drops partners past
        # the last lane), no work in the tasks: pure dependence overhead
        dict(name="fft_300x100", kind="graph", pattern="fft", W=300, T=100, n=256, rounds=0, shape="default"),
        # a dynamic dispatch of the comparators' graph through the ready queue
        dict(name="random_1024x50_queue", kind="graph", pattern="random", W=1024, T=50, n=256, rounds=0,
             shape="queue"),
        # large payloads (64 KiB), one workgroup per task: the bandwidth end
        dict(name="stencil_192x40_n16384", kind="graph", pattern="stencil", W=192, T=40, n=16384, rounds=4,
             shape="workgroup"),
        # tasks that compute for tens of microseconds: the granularity sweep
        dict(name="tree_1024x60_r1024", kind="graph", pattern="tree", W=1024, T=60, n=256, rounds=1024,
             shape="default"),
        # the benchmark's headline step: five patterns of 1024 x 1000 tasks
        dict(name="five_patterns_1024x1000", kind="steps", W=1024, T=1000, n=256, rounds=0, shape="column"),
        # a slice of the uneven batch (widths 8-512, steps 8-256, five payload
        # sizes, log-normal rounds) in one launch
        dict(name="batch_48_uneven", kind="batch", graphs=48, manifest=1, shape="balanced"),
        # an implicit program of the size a serving request has
        dict(name="halo_32x32", kind="halo", P=32, S=256, iters=32, rounds=64, shape="default"),
        # the implicit benchmark program, 65,536 tasks on 2^24 elements
        dict(name="halo_1024x64", kind="halo", P=1024, S=16384, iters=64, rounds=64, shape="gang"),
        # inference of that program's 6.25 million dependences
        dict(name="infer_1024x64", kind="infer", P=1024, S=16384, iters=64, alloc=False),
        # inference of a program with uneven regions and few conflicts per task
        dict(name="regions_30000", kind="regions", tasks=30000, subregions=3001, reads=3),
        # a burst of serving requests, explicit and implicit mixed
        dict(name="serve_48", kind="serve", requests=48, manifest=3, max_tasks=1 << 15),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random):
    kind = rng.choice(["graph", "graph", "graph", "steps", "batch", "halo", "halo", "infer", "infer", "regions",
                       "serve"])
    if kind == "graph":
        n = rng.choice([64, 128, 256, 512, 1024, 4096, 16384])
        W = _log_int(rng, 8, 1024)
        T = _log_int(rng, 8, 1000)
        T = max(2, min(T, (1 << 27) // (n * W)))  # at most half a gigabyte of payloads
        rounds = rng.choice([0, 0, 4, 16, 64, 256, 1024])
        while rounds and n * W * T * rounds > 1 << 34:
            rounds //= 4
        shape = "workgroup" if n >= 4096 else rng.choice(["default", "default", "column", "queue"])
        return dict(kind=kind, pattern=rng.choice(wl.PATTERNS), W=W, T=T, n=n, rounds=rounds, shape=shape)
    if kind == "steps":
        return dict(kind=kind, W=_log_int(rng, 64, 1024), T=_log_int(rng, 50, 400), n=rng.choice([64, 256]), rounds=0,
                    shape="column")
    if kind == "batch":
        return dict(kind=kind, graphs=_log_int(rng, 8, 48), manifest=rng.randrange(1, 1000), shape="balanced")
    if kind == "halo":
        if rng.random() < 0.5:  # request-sized, one wavefront per task
            return dict(kind=kind, P=_log_int(rng, 8, 128), S=256, iters=_log_int(rng, 8, 128),
                        rounds=rng.choice([0, 16, 64, 128]), shape="default")
        return dict(kind=kind, P=_log_int(rng, 128, 1024), S=rng.choice([4096, 10000, 16384]),
                    iters=_log_int(rng, 8, 64), rounds=rng.choice([16, 64]), shape="gang")
    if kind == "infer":
        return dict(kind=kind, P=_log_int(rng, 8, 1024), S=rng.choice([256, 1000, 16384]), iters=_log_int(rng, 4, 64),
                    alloc=rng.random() < 0.5)
    if kind == "regions":
        tasks = _log_int(rng, 500, 30000)
        return dict(kind=kind, tasks=tasks, subregions=max(8, tasks // rng.choice([5, 10, 20])), reads=rng.choice([1, 3, 6]))
    return dict(kind=kind, requests=_log_int(rng, 4, 48), manifest=rng.randrange(1, 1000), max_tasks=1 << 15)


# ----------------------------------------------------------------- inputs

class _Batch:
    """A batch handle that is destroyed with its state."""

    def __init__(self, graphs, cfg):
        self.handle = tg.tg_batch_create([g.handle for g in graphs], cfg)

    def __del__(self):
        tg.tg_batch_destroy(self.handle)


class _Server:
    def __init__(self, budget):
        self.handle = tg.tg_server_create(budget)

    def __del__(self):
        tg.tg_server_destroy(self.handle)


def _cfg(shape):
    s = SHAPES[shape]
    return None if s is None else tg.make_config(**s)


def _explicit(case, seed):
    return wl.pattern_graph(case["pattern"], case["W"], case["T"], seed=seed, n=case["n"], rounds=case["rounds"])


def _halo(case, seed):
    return wl.halo_graph(case["P"], case["S"], case["iters"], seed=seed, rounds=case.get("rounds", 0))


def _first(case, seed):
    """The subregion every sweep of an inferred program starts with."""
    return int(np.random.default_rng([seed, case["P"], case["iters"]]).integers(0, case["P"]))


def _infer_program(case, seed):
    """Requirements of the halo program with its sweeps starting at _first
    (the tasks of a sweep in cyclic order): req_ptr, lo, hi, priv, space."""
    ig, P = _halo(case, seed), case["P"]
    k = np.arange(ig.N, dtype=np.int64)
    old = k - k % P + (k + _first(case, seed)) % P  # the task of the plain program at place k
    beg = ig.req_ptr.astype(np.int64)
    cnt = np.diff(beg)[old]
    ptr = np.zeros(ig.N + 1, np.int64)
    ptr[1:] = np.cumsum(cnt)
    at = np.repeat(beg[old] - ptr[:-1], cnt) + np.arange(ptr[-1])
    return ptr, ig.lo[at], ig.hi[at], ig.priv[at], ig.space


def _batch_specs(case, seed):
    specs = wl.batch_manifest(case["graphs"], seed=case["manifest"])
    return [wl.pattern_graph(s.pattern, s.W, s.T, seed=(seed << 16) + i, n=s.n, rounds=s.rounds)
            for i, s in enumerate(specs)]


def _requests(case, seed):
    reqs = wl.serving_manifest(case["requests"], seed=case["manifest"], max_tasks=case["max_tasks"])
    for i, r in enumerate(reqs):
        r.seed = (seed << 16) + i
    return reqs


def _regions(case, seed):
    """Uneven subregions; task k writes one interval of a random subregion and
    reads one interval of each of `reads` other subregions (cyclic offsets
    from its own, so a task's intervals never overlap).  Returns (req_ptr,
    lo, hi, priv, sub, space): priv 2 = read-write, 1 = read-only; sub is the
    subregion of each interval."""
    rng = np.random.default_rng([seed, case["tasks"], case["subregions"]])
    N, P, K = case["tasks"], case["subregions"], min(case["reads"], case["subregions"] - 1)
    size = rng.integers(200, 3000, P)
    start = np.zeros(P + 1, np.int64)
    start[1:] = np.cumsum(size)
    own = rng.integers(0, P, N)
    off = np.argsort(rng.random((N, min(P - 1, 12))), axis=1)[:, :K] + 1  # distinct, nonzero, below P
    sub = np.concatenate([own[:, None], (own[:, None] + off) % P], axis=1)  # (N, 1 + K)
    a = (rng.random(sub.shape) * 0.5 * size[sub]).astype(np.int64)
    ln = 1 + (rng.random(sub.shape) * 0.5 * (size[sub] - 1)).astype(np.int64)
    lo = start[sub] + a
    hi = np.minimum(lo + ln, start[sub + 1])
    priv = np.ones(sub.shape, np.uint32)
    priv[:, 0] = 2
    req_ptr = np.arange(N + 1, dtype=np.uint64) * np.uint64(1 + K)
    return req_ptr, lo.reshape(-1), hi.reshape(-1), priv.reshape(-1), sub.reshape(-1), int(start[-1])


def _request_form(x):
    """A graph as the benchmark's batch and serving legs run it: implicit ones
    on their reduced dependences, explicit ones reusing payload memory."""
    if isinstance(x, wl.ImplicitGraph):
        g = tg.graph_from_implicit(x)
        tg.tg_graph_reduce_edges(g.handle)
        return g
    return tg.graph_from_explicit(x, retention=tg.TG_KEEP_SINKS)


def _halo_edges(P, iters):
    # any two tasks of one subregion, and any two of neighbouring subregions
    return P * iters * (iters - 1) // 2 + (P - 1) * iters * iters


def _col_capacity(case):
    """Successor entries a program reserves: all pairs that may conflict."""
    if case["kind"] == "infer":
        return _halo_edges(case["P"], case["iters"])
    return int(case["tasks"] * (case["tasks"] / case["subregions"] * (0.5 + case["reads"]) + 8))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "graph":
        g = tg.graph_from_explicit(_explicit(case, seed))
        return dict(kind=kind, g=g, cfg=_cfg(case["shape"]), last=case["W"] * case["T"] - 1)
    if kind == "steps":
        gs = [tg.graph_from_explicit(_explicit(dict(case, pattern=p), seed)) for p in wl.PATTERNS]
        return dict(kind=kind, batch=_Batch(gs, _cfg(case["shape"])), graphs=gs)
    if kind == "batch":
        gs = [_request_form(x) for x in _batch_specs(case, seed)]
        return dict(kind=kind, batch=_Batch(gs, _cfg(case["shape"])), graphs=gs)
    if kind == "halo":
        g = tg.graph_from_implicit(_halo(case, seed))
        if case["shape"] == "gang":  # the benchmark runs it on the reduced dependences
            tg.tg_graph_reduce_edges(g.handle)
        return dict(kind=kind, g=g, cfg=_cfg(case["shape"]), space=case["P"] * case["S"])
    if kind == "serve":
        gs = [_request_form(wl.build_request(r)) for r in _requests(case, seed)]
        return dict(kind=kind, server=_Server(64 << 30), graphs=gs)
    if kind == "infer":
        req_ptr, lo, hi, priv, space = _infer_program(case, seed)
    else:
        req_ptr, lo, hi, priv, _, space = _regions(case, seed)
    N = req_ptr.size - 1
    reqs = tg.reqs_array(lo, hi, priv)
    cap = _col_capacity(case)
    return dict(kind=kind, N=N, M=int(reqs.size), space=space, cap=cap, alloc=case.get("alloc", True),
                req_ptr=torch.from_numpy(req_ptr.astype(np.int64)).cuda(),
                reqs=torch.from_numpy(reqs.view(np.uint8).copy()).cuda(),
                row_ptr=torch.zeros(N + 1, dtype=torch.int64, device="cuda"),
                col=torch.zeros(max(cap, 1), dtype=torch.int32, device="cuda"))


def run(state):
    """The results a program reads: every task's digest (a sum over all words
    of its payload), the shared array of an implicit program, the last task's
    payload.  Payloads stay on the device between tasks by design and reach
    the host one task at a time, so a program that runs a whole graph does not
    read them all."""
    kind = state["kind"]
    if kind == "graph":
        h = state["g"].handle
        tg.tg_graph_execute(h, state["cfg"])
        return dict(digests=tg.tg_graph_read_digests(h), last=tg.tg_graph_read_payload(h, state["last"], state["g"].n))
    if kind in ("steps", "batch"):
        b = state["batch"].handle
        tg.tg_batch_execute(b)
        tg.tg_batch_wait(b)
        return [tg.tg_graph_read_digests(g.handle) for g in state["graphs"]]
    if kind == "halo":
        h = state["g"].handle
        tg.tg_graph_execute(h, state["cfg"])
        return dict(digests=tg.tg_graph_read_digests(h), data=tg.tg_graph_read_data(h, 0, state["space"]))
    if kind == "serve":
        srv = state["server"].handle
        tickets = [tg.tg_server_submit(srv, g.handle) for g in state["graphs"]]
        for t in tickets:
            tg.tg_server_wait(srv, t)
        return [tg.tg_graph_read_digests(g.handle) for g in state["graphs"]]
    infer = tg.tg_infer_dag if state["alloc"] else tg.tg_infer_dag_noalloc
    e = infer(state["N"], state["req_ptr"], state["reqs"], state["M"], state["space"], state["row_ptr"],
              state["col"], state["cap"])
    return dict(row_ptr=state["row_ptr"], col=state["col"], edges=e)  # col[:e]; zeros beyond


# -------------------------------------------------------------- work

def _graph_work(N, E, n, rounds):
    """Every payload written once and (with successors) read once, every edge
    and digest touched once; the mix and the sums over predecessors."""
    return dict(bytes=8 * N * n + 4 * N + 4 * E, flops=N * n * ROUND_OPS * rounds + E * n + 2 * N * n)


def _pattern_edges(pattern, W, T):
    per = {"none": 0, "stencil": 3, "fft": 2, "tree": 1, "random": 5}[pattern]
    return per * W * (T - 1)


def _halo_work(P, S, iters, rounds):
    # the array written at the start and once per sweep, read once per sweep;
    # halos of 32 elements on average
    return dict(bytes=4 * P * S * (1 + 2 * iters) + 4 * P * iters,
                flops=P * S * iters * (ROUND_OPS * rounds + 2) + 64 * P * iters)


def _add(*works):
    return dict(bytes=sum(w["bytes"] for w in works), flops=sum(w["flops"] for w in works))


def work(case):
    kind = case["kind"]
    if kind == "graph":
        return _graph_work(case["W"] * case["T"], _pattern_edges(case["pattern"], case["W"], case["T"]), case["n"],
                           case["rounds"])
    if kind == "steps":
        return _add(*(work(dict(case, kind="graph", pattern=p)) for p in wl.PATTERNS))
    if kind == "batch":
        specs = wl.batch_manifest(case["graphs"], seed=case["manifest"])
        return _add(*(_graph_work(s.W * s.T, _pattern_edges(s.pattern, s.W, s.T), s.n, s.rounds) for s in specs))
    if kind == "halo":
        return _halo_work(case["P"], case["S"], case["iters"], case["rounds"])
    if kind == "serve":
        return _add(*(_graph_work(r.W * r.T, _pattern_edges(r.pattern, r.W, r.T), r.n, r.rounds)
                      if r.mode == "explicit" else _halo_work(r.P, 256, r.iters, r.rounds)
                      for r in _requests(case, 0)))
    if kind == "infer":
        N = case["P"] * case["iters"]
        M = 3 * N - 2 * case["iters"]
        E = _halo_edges(case["P"], case["iters"])
    else:
        N, per = case["tasks"], case["tasks"] / case["subregions"]
        M = N * (1 + case["reads"])
        E = int(N * per * (0.5 + case["reads"]) * 0.6)  # about 0.6 of the pairs in a subregion meet
    return dict(bytes=REQ_BYTES * M + 16 * (N + 1) + 4 * E, flops=4 * E + 4 * M)


def tolerance(case):
    return "exact"


# -------------------------------------------------------------- reference

def _sm64(z):
    with np.errstate(over="ignore"):
        z = z + np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))


def _h32(seed, stream, idx):
    key = _sm64(np.array([(seed ^ (stream << 32)) & 0xFFFFFFFFFFFFFFFF], np.uint64))[0]
    return (_sm64(idx.astype(np.uint64) ^ key) & np.uint64(0xFFFFFFFF)).astype(np.uint32)


def _mix(x, rounds):
    for _ in range(rounds):
        x = x ^ (x << np.uint32(13))
        x = x ^ (x >> np.uint32(17))
        x = x ^ (x << np.uint32(5))
        x = x * np.uint32(0x9E3779B1) + np.uint32(0x7F4A7C15)
    return x


def _exact_graph(eg):
    """Digests and the last task's payload, one timestep at a time.  A sum
    over predecessors is the difference of a running sum along the step's
    predecessor rows, mod 2^32."""
    N, n, W = eg.N, eg.n, eg.W
    digests = np.zeros(N, np.uint32)
    k = np.arange(n, dtype=np.uint64)
    weights = (2 * k + 1).astype(np.uint32)
    out = None
    for t in range(eg.T):
        ids = np.arange(t * W, (t + 1) * W, dtype=np.uint64)
        beg, end = eg.pred_ptr[ids].astype(np.int64), eg.pred_ptr[ids + np.uint64(1)].astype(np.int64)
        if end[-1] == beg[0]:
            x = _h32(eg.seed, 1, (ids[:, None] << np.uint64(16)) | k[None, :])
        else:
            rows = out[eg.preds[beg[0]:end[-1]].astype(np.int64) - (t - 1) * W]
            x = np.add.reduceat(rows, beg - beg[0], axis=0, dtype=np.uint32)
        out = _mix(x ^ ids.astype(np.uint32)[:, None], eg.rounds)
        digests[t * W:(t + 1) * W] = (out * weights[None, :]).sum(axis=1, dtype=np.uint32)
    return digests, out[-1].copy()


def _exact_halo(ig):
    A = _h32(ig.seed, 2, np.arange(ig.space, dtype=np.uint64))
    digests = np.zeros(ig.N, np.uint32)
    w = 2 * np.arange(ig.S, dtype=np.uint32) + np.uint32(1)
    for t in range(ig.N):
        a, b = int(ig.req_ptr[t]), int(ig.req_ptr[t + 1])
        c = np.uint32(0)
        for i in range(a, b):
            if ig.priv[i] == 1:
                c = np.uint32((int(c) + int(A[int(ig.lo[i]):int(ig.hi[i])].sum(dtype=np.uint64))) & 0xFFFFFFFF)
        for i in range(a, b):
            if ig.priv[i] == 2:
                lo, hi = int(ig.lo[i]), int(ig.hi[i])
                A[lo:hi] = _mix(A[lo:hi] ^ c ^ np.uint32(t), ig.rounds)
                digests[t] = (A[lo:hi] * w).sum(dtype=np.uint32)
    return digests, A


def _rows(N, src, dst, cap):
    order = np.lexsort((dst, src))
    src, dst = src[order], dst[order]
    row_ptr = np.zeros(N + 1, np.int64)
    row_ptr[1:] = np.cumsum(np.bincount(src, minlength=N))
    col = np.zeros(max(cap, 1), np.int32)
    col[:dst.size] = dst
    return dict(row_ptr=torch.from_numpy(row_ptr), col=torch.from_numpy(col), edges=int(dst.size))


def _exact_halo_dag(case, seed):
    """Halos are at least one and at most S elements wide, so two tasks
    conflict exactly when their subregions are equal or neighbours."""
    P, iters, first = case["P"], case["iters"], _first(case, seed)
    N = P * iters
    j = np.arange(N, dtype=np.int64)
    sub = (j + first) % P
    src, dst = [], []
    for d in range(iters):
        for ds in (-1, 0, 1):
            to = j - j % P + d * P + (sub + ds - first) % P
            ok = (sub + ds >= 0) & (sub + ds < P) & (to < N) & (to > j)
            src.append(j[ok])
            dst.append(to[ok])
    return _rows(N, np.concatenate(src), np.concatenate(dst), _col_capacity(case))


def _exact_regions(case, seed):
    """All pairs of intervals of each subregion."""
    req_ptr, lo, hi, priv, sub, _ = _regions(case, seed)
    N = case["tasks"]
    task = np.repeat(np.arange(N, dtype=np.int64), np.diff(req_ptr.astype(np.int64)))
    order = np.argsort(sub, kind="stable")
    bounds = np.searchsorted(sub[order], np.arange(case["subregions"] + 1))
    keys = []
    for s in range(case["subregions"]):
        m = order[bounds[s]:bounds[s + 1]]
        hit = (lo[m][:, None] < hi[m][None, :]) & (lo[m][None, :] < hi[m][:, None])
        hit &= (priv[m][:, None] == 2) | (priv[m][None, :] == 2)
        hit &= task[m][:, None] < task[m][None, :]
        x, y = np.nonzero(hit)
        keys.append(task[m][x] * N + task[m][y])
    keys = np.unique(np.concatenate(keys))
    return _rows(N, keys // N, keys % N, _col_capacity(case))


def exact(case, seed):
    kind = case["kind"]
    if kind == "graph":
        if work(case)["flops"] > 4e9:
            return None
        digests, last = _exact_graph(_explicit(case, seed))
        return dict(digests=digests, last=last)
    if kind == "halo":
        if work(case)["flops"] > 4e9 or case["P"] * case["iters"] > 100000:
            return None
        digests, data = _exact_halo(_halo(case, seed))
        return dict(digests=digests, data=data)
    if kind == "infer":
        return _exact_halo_dag(case, seed)
    if kind == "regions":
        return _exact_regions(case, seed)
    if kind in ("batch", "steps", "serve") and work(case)["flops"] > 4e9:
        return None
    if kind == "serve":
        out = []
        for x in map(wl.build_request, _requests(case, seed)):
            out.append(_exact_halo(x)[0] if isinstance(x, wl.ImplicitGraph) else _exact_graph(x)[0])
        return out
    graphs = (_batch_specs(case, seed) if kind == "batch" else
              [_explicit(dict(case, pattern=p), seed) for p in wl.PATTERNS])
    return [_exact_graph(x)[0] for x in graphs]
