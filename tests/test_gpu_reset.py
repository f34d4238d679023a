"""What a launch starts from: the initial arrays of every implicit graph of a
batch, however they are mixed with explicit ones and with each other's sizes,
and the ready queue with fewer, as many and more sources than shards, after a
launch that left its slots filled.  Several launches of one layout, each
bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2508_16522_amd import taskgraph as tg
from paper_2508_16522_amd import workloads as wl
from tests.gpu_util import check_explicit, oracle_explicit

pytestmark = pytest.mark.gpu

SHAPES = {"lists": dict(mapping=1), "queue": dict(mapping=1, dispatch=tg.TG_DISPATCH_QUEUE),
          "queue, workgroups": dict(mapping=2, wg_waves=2, dispatch=tg.TG_DISPATCH_QUEUE)}


def readers(space, seed):
    """Two tasks that read the whole array and write its halves: every word's
    initial value shows in the result."""
    h = space // 2
    return wl.ImplicitGraph(N=2, req_ptr=np.array([0, 2, 4], np.uint64), lo=np.array([0, h, h, 0], np.uint64),
                            hi=np.array([h, space, space, h], np.uint64), priv=np.array([1, 2, 1, 2], np.uint32),
                            space=space, rounds=1, seed=seed)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("sources", [1, 7, 8, 9, 300])
def test_launch_state(gpu, sources, shape):
    egs = [wl.pattern_graph("none", sources - 6, 1, seed=7) if sources > 6 else None,
           wl.pattern_graph("stencil", 1, 5, seed=8)]
    igs = [readers(s, seed=s) for s in (2, 3, 255, 257, 70001)] if sources > 6 else []
    graphs = []
    for k in range(max(len(igs), 2)):
        if k < len(igs):
            graphs.append(igs[k])
        if k < 2 and egs[k] is not None:
            graphs.append(egs[k])
    gs = [(tg.graph_from_implicit if isinstance(x, wl.ImplicitGraph) else tg.graph_from_explicit)(x) for x in graphs]
    b = tg.tg_batch_create([g.handle for g in gs], tg.make_config(**SHAPES[shape]))
    try:
        for _ in range(3):
            tg.tg_batch_execute(b)
            tg.tg_batch_wait(b)
            for g, x in zip(gs, graphs):
                if isinstance(x, wl.ImplicitGraph):
                    ref = oracle.implicit_program_order(x.N, x.req_ptr, x.lo, x.hi, x.priv, x.rounds, x.space, seed=x.seed)
                    assert np.array_equal(tg.tg_graph_read_data(g.handle, 0, x.space), ref["A"])
                    assert np.array_equal(tg.tg_graph_read_digests(g.handle), ref["digest"])
                else:
                    check_explicit(g, x, oracle_explicit(x), payload_sample=8)
    finally:
        tg.tg_batch_destroy(b)
