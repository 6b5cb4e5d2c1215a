"""The routing analytics where their kernels' work splits: token counts around a rank
workgroup (16 tokens, entropies compared four at a time), an entropy workgroup (64 tokens, 4
to a wave) and the batches of the load and summary kernels (12 x 1024 pairs, 6 x 1024
tokens), candidate counts 1 to 16, ties.  Same reference and tolerance as
tests/test_routing_stats.py."""
import pytest

from tests import test_routing_stats as base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 3, 17, 63, 64, 65, 1023, 1025, 6145])
@pytest.mark.parametrize("E,K,Kb,ratio,levels", [(64, 16, 0, 0.3, None), (16, 1, 1, 1.0, None), (33, 7, 1, 0.6, 8)])
def test_edges(T, E, K, Kb, ratio, levels):
    base.test_gpu_routing_stats_match_oracle(T, E, K, Kb, ratio, levels)
