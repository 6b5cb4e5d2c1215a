"""Correlation of token entropies with keep counts where its kernel's sums can go wrong: one token,
all tokens keeping the same number, every keep count from 0 to K = 16, equal entropies, token counts
around a batch of loads.  Protocol of tests/test_routing_stats.py: scipy's Spearman in 64 bits."""
import pytest
import torch
from scipy import stats as sps

from paper_2604_08133_amd import binding as B, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,K,kind", [(1, 4, "mixed"), (700, 4, "same"), (1023, 16, "mixed"), (1025, 16, "mixed"),
                                      (6143, 6, "mixed"), (6145, 6, "mixed"), (3000, 8, "ties")])
def test_token_correlation(T, K, kind):
    E = 20
    scores = synth.make_scores(T, E, seed=53)
    if kind == "ties":
        scores = scores[torch.arange(T) % 7].contiguous()
    g = torch.Generator().manual_seed(54)
    keep = torch.full((T,), 2) if kind == "same" else torch.randint(0, K + 1, (T,), generator=g)
    desc = B.make_desc(T, 64, E, 64, K, 0, T * K, "f32")
    top, ids = scores.topk(K, dim=1)
    out = B.allocmoe_routing_stats(desc, scores.cuda(), ids.int().cuda(), top.contiguous().cuda(), keep.int().cuda())
    got = float(out["metrics"][4])
    if T == 1 or kind == "same":
        assert got == 0.0   # one side constant
        return
    want = float(sps.spearmanr(out["token_entropy"].cpu().double().numpy(), keep.numpy()).statistic)
    assert abs(got - want) <= 1e-6   # exact integer sums, one rounding to fp32
