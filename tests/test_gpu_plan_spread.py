"""Selection and dispatch as a sequence of launches: ties at the threshold that are split among the tokens of
several workgroups and of several groups of histograms (up to 16384 tokens a group is a workgroup's 1024
tokens, beyond it a sixteenth of all), and pools of every number of entries a token, whose loads overlap or end
inside, at rows of any 4-byte boundary.  Bit for bit against the oracle from the same scores."""
import pytest

from paper_2604_08133_amd import synth
from tests.test_gpu_route_dispatch import assert_same, gpu_route_dispatch, oracle_route_dispatch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,K,Kb,levels", [(4096, 8, 2, 1, 8), (4097, 64, 8, 0, 64), (8193, 33, 5, 2, 16), (9216, 20, 16, 0, 32),
                                             (16384, 16, 3, 0, 16), (16385, 16, 3, 1, 16), (33000, 12, 4, 0, 0),
                                             (33000, 12, 4, 0, 16), (50001, 6, 2, 0, 4), (4100, 20, 4, 0, 16),
                                             (4100, 20, 5, 0, 16), (4100, 20, 7, 0, 0), (4100, 20, 9, 0, 16),
                                             (4100, 20, 10, 1, 16), (4100, 20, 12, 1, 0), (4100, 20, 13, 0, 16),
                                             (4100, 20, 15, 0, 0), (4100, 20, 3, 0, 8), (16385, 16, 15, 2, 32),
                                             (20001, 10, 5, 0, 8)])
def test_ties_across_workgroups(T, E, K, Kb, levels):
    scores = synth.make_scores(T, E, seed=61, quantize_levels=levels or None)
    n_pool = T * (K - Kb)
    for extra in (1, n_pool // 3, n_pool // 2 + 1, n_pool - 1):
        args = (scores, K, Kb, T * Kb + extra)
        print(f"T={T} K={K} Kb={Kb} levels={levels} extra={extra}", flush=True)
        assert_same(gpu_route_dispatch(*args), oracle_route_dispatch(*args), extra)
