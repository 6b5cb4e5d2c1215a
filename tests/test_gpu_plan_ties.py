"""Selection of the one-launch plan kernel where much of the pool falls into one bin and the bin's own
range is measured: one crowd of equal keys (padding tokens), several crowds, keys one unit in the
last place apart, a crowd beside keys far away.  Every block size of the kernel, the threshold below,
inside and above the crowd.  Bit for bit against the oracle run from the same scores."""
import pytest
import torch

from paper_2604_08133_amd import synth
from tests.test_gpu_route_dispatch import assert_same, gpu_route_dispatch, oracle_route_dispatch

pytestmark = pytest.mark.gpu


def crowded(T, E, kind):
    scores = synth.make_scores(T, E, seed=61)
    row = torch.full((E,), 1.0 / E)
    share = {"half": 0.5, "most": 0.9, "all": 1.0}.get(kind, 0.75)
    crowd = (torch.arange(T) * 7919 % T) < share * T
    if kind == "two":   # two crowds of different keys
        scores[crowd] = torch.where((torch.arange(T) % 2 == 0)[crowd][:, None], row, row / 3)
    elif kind == "close":   # 512 neighbouring fp32 values
        bits = row.view(torch.int32)[None, :] + (torch.arange(T)[:, None] * 31 + torch.arange(E)[None, :]) % 512
        scores[crowd] = bits.to(torch.int32).view(torch.float32)[crowd]
    elif kind == "far":   # the others at both ends of the exponent range, infinity and zero
        scores[crowd] = row
        scores[~crowd] = torch.tensor([0.0, 1e-40, 3e38, float("inf")])[torch.arange(T * E).reshape(T, E)[~crowd] % 4]
    else:
        scores[crowd] = row
    return scores.contiguous()


@pytest.mark.parametrize("kind", ["half", "most", "all", "two", "close", "far"])
@pytest.mark.parametrize("T,K,Kb", [(200, 4, 0), (256, 16, 0), (512, 8, 1), (1500, 6, 0), (6000, 8, 1)])
def test_crowded_bins(T, K, Kb, kind):
    scores = crowded(T, 64, kind)
    n_pool = T * (K - Kb)
    for extra in sorted({1, n_pool // 10, n_pool // 2, 9 * n_pool // 10, n_pool - 1}):
        args = (scores, K, Kb, T * Kb + extra)
        # (without a workspace one workgroup selects whatever the size)
        assert_same(gpu_route_dispatch(*args, select_ws=False), oracle_route_dispatch(*args), (kind, extra))
