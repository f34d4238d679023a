"""Every in-degree and out-degree around the sizes at which a task changes
path (five predecessors loaded at once, six held in its record; eight
successors held there; one or several chunks of a payload per lane), in each
executor, with and without diagnostics, against the oracle (bit-exact)."""
import numpy as np
import pytest

from paper_2508_16522_amd import taskgraph as tg
from paper_2508_16522_amd import workloads as wl
from tests.gpu_util import check_explicit, oracle_explicit, run

pytestmark = pytest.mark.gpu

SHAPES = {
    "lists": dict(mapping=1),
    "one worker": dict(mapping=1, workers=1),
    "columns": dict(mapping=1, schedule=tg.TG_SCHED_COLUMN, window=1),
    "workgroup": dict(mapping=2, wg_waves=2),
    "workgroup of three": dict(mapping=2, wg_waves=3),  # chunks that do not divide a payload
    "gang": dict(mapping=3, wg_waves=2, gang=2),
    "queue": dict(mapping=1, dispatch=tg.TG_DISPATCH_QUEUE),
    "queue, workgroup": dict(mapping=2, wg_waves=2, dispatch=tg.TG_DISPATCH_QUEUE),
}


def fan_graph(n, rounds):
    """Three layers: 70 sources; tasks with 1 .. 13 and 66 of them as
    predecessors; and 70 tasks that read 2 or 6 of the middle ones, so that out-degrees
    run from 0 to 70."""
    lists = [[] for _ in range(70)]
    for k in list(range(1, 14)) + [66]:
        lists.append(list(range(3, 3 + k)))
    for i in range(70):
        lists.append([70 + i % 14, 83] if i % 2 else [70 + (i + d) % 14 for d in range(6)])
    ptr = np.zeros(len(lists) + 1, np.uint64)
    ptr[1:] = np.cumsum([len(x) for x in lists])
    return wl.ExplicitGraph(N=len(lists), pred_ptr=ptr, preds=np.array([p for x in lists for p in x], np.uint32), n=n,
                            rounds=rounds, seed=n)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("n", [64, 128, 256, 512, 2048])
def test_degrees(gpu, n, shape):
    eg = fan_graph(n, 2)
    ref = oracle_explicit(eg)
    g = tg.graph_from_explicit(eg)
    for diag in (0, 1, 0):
        run(g, tg.make_config(diag=diag, **SHAPES[shape]))
        check_explicit(g, eg, ref, payload_sample=70)
