"""The schedule the library chooses for one graph: a graph whose columns would
run independent expensive tasks one after another keeps its parallelism."""
import numpy as np
import pytest

from paper_2508_16522_amd import taskgraph as tg
from paper_2508_16522_amd import workloads as wl
from tests.gpu_util import check_explicit, oracle_explicit

pytestmark = pytest.mark.gpu


def _leaves(steps, leaf_rounds):
    """A chain of empty tasks, each releasing one leaf of `leaf_rounds`."""
    N = 2 * steps
    preds = np.empty(N - 1, np.uint32)  # every task but the first has one
    k = np.arange(N)
    preds[:] = np.where(k % 2 == 1, k - 1, k - 2)[1:]
    ptr = np.concatenate([[0], np.arange(N)]).astype(np.uint64)
    rounds = np.where(k % 2 == 1, leaf_rounds, 0).astype(np.uint32)
    return wl.ExplicitGraph(N=N, pred_ptr=ptr, preds=preds, n=256, rounds=rounds)


def _build(eg):
    g = tg.Graph(tg.tg_graph_create(tg.TG_EXPLICIT, eg.n, 0, eg.seed), tg.TG_EXPLICIT, eg.n)
    tg.tg_task_add_many(g.handle, eg.pred_ptr, eg.preds, eg.rounds)
    tg.tg_graph_finalize(g.handle)
    return g


def _time(g, cfg):
    for _ in range(4):
        tg.tg_graph_execute(g.handle, cfg)
        tg.tg_graph_wait(g.handle)
    return min(tg.tg_graph_kernel_times(g.handle, 3))


@pytest.mark.parametrize("mapping", [tg.TG_MAP_WAVE, tg.TG_MAP_WORKGROUP])
def test_leaves_of_a_chain_run_side_by_side(gpu, mapping):
    eg = _leaves(200, 1024)
    g = _build(eg)
    level = _time(g, tg.make_config(mapping=mapping, schedule=tg.TG_SCHED_LEVEL))
    column = _time(g, tg.make_config(mapping=mapping, schedule=tg.TG_SCHED_COLUMN))
    own = _time(g, tg.make_config(mapping=mapping))
    # one after another the leaves take 200 times one of them
    assert column > 3 * level, (column, level)
    assert own < 1.5 * level, (own, level)
    ref = oracle_explicit(eg)
    check_explicit(g, eg, ref)


def test_the_choice_follows_the_rounds(gpu):
    """Uneven rounds set to one value: the graph runs on the order that suits it
    now, with the results of its new rounds."""
    eg = _leaves(40, 512)
    g = _build(eg)
    tg.tg_graph_execute(g.handle)
    check_explicit(g, eg, oracle_explicit(eg))
    for r in (3, 0):
        tg.tg_graph_set_rounds(g.handle, r)
        eg.rounds = r
        tg.tg_graph_execute(g.handle)
        tg.tg_graph_execute(g.handle)
        check_explicit(g, eg, oracle_explicit(eg))
