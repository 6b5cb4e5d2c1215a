"""Dispatch on several workgroups of one launch: above 1536 tokens each forms words for a run of 64-token batches and counts
the pairs of the others (up to 8 candidates a token), so runs that end inside a batch, workgroups without one, tokens that keep nothing,
one expert that takes all or is in every token, an id that a token repeats (one row, as in a word), and one that fills
the places behind the kept candidates.  Whole numbers, so bit for bit."""
import pytest
import torch

from paper_2604_08133_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def on_gpu(ids, cnt, E, budget):
    T, K = ids.shape
    desc = B.make_desc(T, 64, E, 64, K, 0, budget, "f32")
    offs = torch.empty((E + 1,), dtype=torch.int32, device=DEV)
    row_token = torch.full((budget,), -7, dtype=torch.int32, device=DEV)
    row_rank = torch.full((budget,), -7, dtype=torch.int32, device=DEV)
    inv_row = torch.empty((T, K), dtype=torch.int32, device=DEV)
    ws = torch.empty(B.allocmoe_workspace_layout(desc).scores, dtype=torch.uint8, device=DEV)
    B.allocmoe_dispatch(desc, ids.to(DEV), cnt.to(DEV), offs, row_token, row_rank, inv_row, ws)
    torch.cuda.synchronize()
    return offs.cpu(), row_token.cpu(), row_rank.cpu(), inv_row.cpu()


def in_order(ids, cnt, E):
    """Rows by expert, then token; a token's later repeat of an expert shares the row of the first."""
    T, K = ids.shape
    kept = torch.arange(K)[None, :] < cnt[:, None]
    pair = torch.zeros((E, T), dtype=torch.int64)
    pair[ids[kept].long(), torch.arange(T)[:, None].expand(T, K)[kept]] = 1
    row_of = (pair.flatten().cumsum(0) - 1).view(E, T)
    offs = torch.cat([torch.zeros(1, dtype=torch.int64), pair.sum(1).cumsum(0)]).int()
    inv = torch.where(kept, row_of[ids.long(), torch.arange(T)[:, None]], torch.tensor(-1)).int()
    row_token = torch.full((int(offs[-1]),), -7, dtype=torch.int32)
    row_rank = row_token.clone()
    for j in range(K):   # of pairs that share a row the later one's rank stays
        at = inv[kept[:, j], j].long()
        row_token[at] = torch.nonzero(kept[:, j])[:, 0].int()
        row_rank[at] = j
    return offs, row_token, row_rank, inv


@pytest.mark.parametrize("T", [513, 1025, 1536, 1537, 1600, 1601, 2047, 2049, 3000, 6143])
@pytest.mark.parametrize("E,K,kind", [(64, 8, "counts"), (64, 16, "counts"), (33, 5, "sparse"), (5, 3, "one"), (9, 7, "repeats"),
                                      (64, 8, "hot"), (33, 6, "filled"), (64, 9, "hot")])
def test_runs_of_batches(T, E, K, kind):
    gen = torch.Generator().manual_seed(T * 131 + E)
    if kind == "repeats":
        ids = torch.randint(0, E, (T, K), generator=gen, dtype=torch.int32)
    else:
        ids = torch.rand((T, E), generator=gen).argsort(1)[:, :K].int().contiguous()
    cnt = torch.randint(0, K + 1, (T,), generator=gen, dtype=torch.int32)
    if kind == "sparse":
        cnt[torch.rand(T, generator=gen) < 0.97] = 0
    if kind == "hot":   # expert 3 is every token's first
        at = (ids == 3).int().argmax(1)
        ids[torch.arange(T), at] = ids[:, 0]
        ids[:, 0] = 3
        cnt.clamp_(min=1)
    if kind == "filled":
        ids = torch.where(torch.arange(K)[None, :] < cnt[:, None], ids, torch.full_like(ids, E - 1))
    if kind == "one":
        ids[:, 0] = 2
        ids[:, 1:] = torch.tensor([0, 4], dtype=torch.int32)
        cnt.fill_(1)
    want = in_order(ids, cnt, E)
    got = on_gpu(ids, cnt, E, max(1, int(cnt.sum())))
    n = int(want[0][-1])
    for w, g, name in zip(want, got, ("offsets", "row_token", "row_rank", "inv_row")):
        assert torch.equal(g[:n] if name.startswith("row") else g, w), (T, kind, name)
