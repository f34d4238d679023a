"""The mix of the task bodies at every vector width it is compiled for (one,
two or four words per lane, and several chunks of four), against the oracle's
written-out rounds (bit-exact)."""
import pytest

from paper_2508_16522_amd import taskgraph as tg
from paper_2508_16522_amd import workloads as wl
from tests.gpu_util import check_explicit, oracle_explicit, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rounds", [0, 1, 2, 7, 8, 9, 63, 257])
@pytest.mark.parametrize("n", [64, 128, 256, 512])
def test_mix_widths(gpu, n, rounds):
    # sources take every 32-bit pattern the hash gives; the second step mixes
    # sums, so both words of a pair differ in all bits
    eg = wl.pattern_graph("stencil", 33, 3, seed=rounds + n, n=n, rounds=rounds)
    ref = oracle_explicit(eg)
    g = tg.graph_from_explicit(eg)
    for cfg in (tg.make_config(mapping=1), tg.make_config(mapping=2, wg_waves=2)):
        run(g, cfg)
        check_explicit(g, eg, ref, payload_sample=32)
