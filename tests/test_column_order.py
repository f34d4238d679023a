"""The column schedule of one graph takes a short cut (a counting sort by
level); next to an empty graph the same graph takes the general path, and both
must give the same lists (CPU)."""
import numpy as np
import pytest

from paper_2508_16522_amd import taskgraph as tg
from paper_2508_16522_amd import workloads as wl


def _graphs():
    rng = np.random.default_rng(0)
    for p in wl.PATTERNS:
        yield p, wl.pattern_graph(p, 37, 9, seed=1)
    yield "dag", wl.random_dag(200, 4, rng)
    yield "one task", wl.random_dag(1, 4, rng)
    yield "chain", wl.pattern_graph("stencil", 1, 70)


@pytest.mark.parametrize("nworkers", [1, 3, 37, 64, 500])
def test_one_graph_equals_the_general_order(tglib, nworkers):
    empty = tg.graph_from_explicit(wl.ExplicitGraph(N=0, pred_ptr=np.zeros(1, np.uint64), preds=np.zeros(0, np.uint32)))
    for name, eg in _graphs():
        g = tg.graph_from_explicit(eg)
        a = tg.tg_emulate_schedule(g.handle, nworkers, 64, 5, tg.TG_SCHED_COLUMN)
        b = tg.tg_emulate_schedule([g.handle, empty.handle], nworkers, 64, 5, tg.TG_SCHED_COLUMN)
        assert a[0] == b[0] == tg.TG_OK, name
        assert np.array_equal(a[1], b[1]) and a[2:] == b[2:], name
