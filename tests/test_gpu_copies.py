"""Reading results back: they come in blocks of 1 MiB through pinned memory,
taken by several threads where there are more than two.  Bit-exact against
the oracle for every remainder, for parts of the array, and for many callers
at once (more than there are blocks)."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle
from paper_2508_16522_amd import taskgraph as tg
from paper_2508_16522_amd import workloads as wl
from tests.gpu_util import run

pytestmark = pytest.mark.gpu

MIB = 1 << 18  # words


def one_sweep(words):
    """The whole array written by 257 tasks of nearly equal length."""
    cut = np.linspace(0, words, 258).astype(np.uint64)
    return wl.ImplicitGraph(N=257, req_ptr=np.arange(258, dtype=np.uint64), lo=cut[:-1].copy(), hi=cut[1:].copy(),
                            priv=np.full(257, 2, np.uint32), space=words, rounds=1, seed=words)


@pytest.mark.parametrize("words", [MIB - 1, MIB, MIB + 1, 2 * MIB + 1, 3 * MIB, 17 * MIB + 3])
def test_blocks(gpu, words):
    import torch
    ig = one_sweep(words)
    ref = oracle.implicit_program_order(ig.N, ig.req_ptr, ig.lo, ig.hi, ig.priv, ig.rounds, ig.space, seed=ig.seed)["A"]
    g = tg.graph_from_implicit(ig)
    run(g)

    def part(lo, hi):
        return np.array_equal(tg.tg_graph_read_data(g.handle, lo, hi), ref[lo:hi])

    assert part(0, words)
    assert part(words - 1, words) and part(words, words)
    assert part(7, words - 5)
    pinned = torch.zeros(words, dtype=torch.int32, pin_memory=True)  # copied to directly
    tg._check(tg.load().tg_graph_read_data(g.handle, pinned.data_ptr(), 0, words), "tg_graph_read_data")
    assert np.array_equal(pinned.numpy().view(np.uint32), ref)
    with ThreadPoolExecutor(12) as ex:
        assert all(ex.map(lambda k: part(k, words - k), range(12)))
