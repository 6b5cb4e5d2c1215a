"""The routing kernel of row-major gates on both sides of its choice of 4 or 16 waves, by hidden
size and by tokens, and above the 2^24 tokens that 16 waves could launch."""
import pytest
import torch

from paper_2604_08133_amd import binding as B

pytestmark = pytest.mark.gpu


def route(X, Wg, K):
    T, d = X.shape
    E = Wg.shape[1]
    desc = B.make_desc(T, d, E, 64, K, 1, T * (K + 1) // 2, X.dtype)
    i32 = dict(dtype=torch.int32, device="cuda")
    scores = torch.empty((T, E), device="cuda")
    ids, keep = torch.empty((T, K), **i32), torch.empty((T,), **i32)
    s = torch.empty((T, K), device="cuda")
    ws = torch.empty(B.allocmoe_workspace_layout(desc).scores, dtype=torch.uint8, device="cuda")
    B.allocmoe_route(desc, X, B.make_weights(Wg=Wg), scores, ids, s, keep, ws)
    return scores, ids, s, keep


def check(X, Wg, K, rows):
    scores, ids, s, keep = route(X, Wg, K)
    assert int(keep.sum()) == X.shape[0] * (K + 1) // 2
    scores, ids, s = scores[rows], ids[rows], s[rows]
    logits = X[rows].double() @ Wg.double()
    # a score's relative error is that of exp(logit): products and sums in fp32, d + 1 roundings
    # of at most sum |x w| each
    bound = float(2 * (X.shape[1] + 8) * 2.0 ** -24 * (X[rows].double().abs() @ Wg.double().abs()).max())
    want = torch.softmax(logits, dim=1)
    assert ((scores.double() - want).abs() <= bound * want + 1e-30).all()
    # the candidates are exact functions of the scores
    top, at = torch.sort(scores, dim=1, descending=True, stable=True)
    assert torch.equal(s, top[:, :K]) and torch.equal(ids.long(), at[:, :K])


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,d", [(7, 256), (7, 257), (8191, 768), (8192, 768), (8192, 769), (65535, 321),
                                 (65536, 832), (65533, 832), (5, 1), (3, 1025)])
def test_both_wave_counts(T, d, dtype):
    if dtype == torch.bfloat16:
        d = (d + 63) // 64 * 64
    g = torch.Generator(device="cuda").manual_seed(T * 7 + d)
    X = torch.randn((T, d), generator=g, device="cuda").to(dtype)
    Wg = (torch.randn((d, 61), generator=g, device="cuda") / d ** 0.5).to(dtype)
    rows = torch.arange(T, device="cuda") if T < 500 else torch.randint(0, T, (500,), generator=g, device="cuda")
    check(X, Wg, 5, rows)


@pytest.mark.parametrize("d", [2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 80, 81, 1000, 1132])
def test_rows_of_a_chunk(d):
    """Gate rows come 16 at a time, the next ones ahead: chunks of 64 that end before, at and behind each step, and
    experts whose rows lie next to memory that holds no number."""
    T, E = 6, 61
    g = torch.Generator(device="cuda").manual_seed(d)
    X = torch.randn((T, d), generator=g, device="cuda")
    room = torch.full((d + 128, E), float("nan"), device="cuda")
    room[64:64 + d] = torch.randn((d, E), generator=g, device="cuda") / d ** 0.5
    check(X, room[64:64 + d], 5, torch.arange(T, device="cuda"))


def test_more_tokens_than_sixteen_waves_can_launch():
    T, d, E = 2 ** 24 + 5, 257, 3
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 3 * T * d * 4:
        pytest.skip("needs 52 GB of device memory")
    # (few distinct rows, so that inputs are quick to make)
    g = torch.Generator(device="cuda").manual_seed(3)
    X = torch.randn((4099, d), generator=g, device="cuda").repeat(T // 4099 + 1, 1)[:T]
    Wg = torch.randn((d, E), generator=g, device="cuda") / d ** 0.5
    rows = torch.cat([torch.arange(0, T, 40009, device="cuda"), torch.arange(T - 9, T, device="cuda")])
    check(X.contiguous(), Wg, 1, rows)
