"""The fp32 expert networks against the same sums in 64 bits: contraction depths around a step and the four
waves' share of steps, columns around a workgroup's 64, rows around the 16-row blocks; sums of few terms and
operands down to the smallest numbers, whose products have to carry all bits of an fp32 product; and operands
and sums that are not finite.

Tolerance: products are exact and a sum of n terms carries at most n roundings of 2^-24, each of a partial sum
that is at most sum |x w|, so n 2^-24 of that bounds it (with 2^-150 for each rounding of a subnormal number). Where H
is compared, twice that: the SwiGLU factor's own error is below 1e-6."""
import pytest
import torch

from paper_2604_08133_amd import binding as B, synth
from paper_2604_08133_amd.layer import DeviceLayer

pytestmark = pytest.mark.gpu


def run_layer(d, I, T, change=None, seed=7):
    w = synth.Workload("f32_parts", T=T, d=d, E=2, I=I, K=2, K_base=1, budget=2 * T, dtype="f32", I_shared=0,
                       I_shared_each=0)
    layer = synth.make_layer(w, seed=seed)
    if change is not None:
        change(layer)
    print(f"d={d} I={I} T={T}", flush=True)
    dev = DeviceLayer(w, layer)
    dev.forward()
    torch.cuda.synchronize()
    mid = {k: v.cpu() for k, v in dev.intermediates().items()}
    offs, rows = mid["expert_offsets"].tolist(), mid["row_token"].long()
    want, bound = torch.empty_like(mid["H"], dtype=torch.float64), torch.empty_like(mid["H"], dtype=torch.float64)
    for e in range(2):
        x = layer["X"][rows[offs[e]:offs[e + 1]]].double()
        a, b = x @ layer["W1"][e].double(), x @ layer["W3"][e].double()
        want[offs[e]:offs[e + 1]] = a * torch.sigmoid(a) * b
        ea, eb = (2 * d * 2.0 ** -24 * (x.abs() @ layer[n][e].double().abs()) for n in ("W1", "W3"))
        # |d silu / da| <= 1.1
        bound[offs[e]:offs[e + 1]] = 1.1 * ea * (b.abs() + eb) + (a * torch.sigmoid(a)).abs() * eb + 1e-6 * want[offs[e]:offs[e + 1]].abs()
    return mid["H"], want, bound, offs


@pytest.mark.parametrize("d,I", [(31, 63), (32, 64), (33, 65), (127, 4), (128, 68), (129, 5), (161, 130), (5, 64)])
@pytest.mark.parametrize("T", [1, 16, 17, 32, 33])
def test_sums(d, I, T):
    H, want, bound, _ = run_layer(d, I, T)
    assert ((H.double() - want).abs() <= bound).all()


def test_error_of_long_sums():
    """2-norm against 64 bits; with fp32 products 4.6e-7 at this depth."""
    H, want, _, _ = run_layer(1206, 200, 96)
    assert float((H.double() - want).norm() / want.norm()) <= 5e-7


@pytest.mark.parametrize("T", [9, 24, 40])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 3.4e38, -3.4e38, 2.0 ** 127])
def test_operands_without_parts(value, T):
    """One weight of expert 0 is `value`: its column as in 32-bit arithmetic, everything else unchanged."""
    k, n = 40, 70

    def change(layer):
        layer["X"][:, k] = torch.where(torch.arange(layer["X"].shape[0]) % 2 == 0, 0.25, -0.5)
        layer["W3"][0, k, n] = value
    H, want, bound, offs = run_layer(100, 132, T, change)
    H, want = H.double(), want.float().double()   # (what overflows 32 bits is infinite)
    finite = torch.isfinite(want)
    assert torch.equal(torch.isnan(H), torch.isnan(want))
    assert torch.equal(H[~finite & ~torch.isnan(want)], want[~finite & ~torch.isnan(want)])
    assert ((H - want).abs()[finite] <= bound[finite]).all()
    others = torch.ones_like(finite)
    others[offs[0]:offs[1], n] = False
    assert finite[others].all() and torch.isfinite(H[others]).all()


def second_half(w, change, seed=7):
    """The layer's (H, O, offsets) and, with a shared expert, (Hs, Os); `change` alters its tensors first."""
    layer = synth.make_layer(w, seed=seed)
    change(layer)
    dev = DeviceLayer(w, layer)
    dev.forward()
    torch.cuda.synchronize()
    mid = dev.intermediates()
    out = [layer, mid["H"].cpu(), mid["O"].cpu(), mid["expert_offsets"].tolist()]
    if w.I_shared:
        desc = dev.desc()
        L, ws = B.allocmoe_workspace_layout(desc), dev.workspace(desc)
        out += [B.ws_view(ws, L.Hs, (w.T, w.I_shared), torch.float32).cpu(),
                B.ws_view(ws, L.Os, (w.T, w.d), torch.float32).cpu()]
    return out


@pytest.mark.parametrize("terms", [1, 2, 4, 512])
@pytest.mark.parametrize("scale", [0, -112, -121, -135])
def test_few_terms_and_small_operands(terms, scale):
    """O = H W2 where H has `terms` columns that are not zero and W2 is of the order of 2^scale."""
    T, d, I = 40, 600, 512
    w = synth.Workload("f32_terms", T=T, d=d, E=2, I=I, K=2, K_base=1, budget=2 * T, dtype="f32")

    def change(layer):
        held = torch.zeros(I, dtype=torch.bool)
        held[torch.arange(terms) * (I // terms)] = True
        for n in ("W1", "W3"):
            layer[n] = layer[n] * held
        layer["W2"] = (layer["W2"].double() * 2.0 ** scale).float()
    print(f"terms={terms} scale={scale}", flush=True)
    layer, H, O, offs = second_half(w, change)
    H, O = H.double(), O.double()
    for e in range(2):
        h, w2 = H[offs[e]:offs[e + 1]], layer["W2"][e].double()
        bound = terms * (2.0 ** -24 * (h.abs() @ w2.abs()) + 2.0 ** -150)
        assert ((O[offs[e]:offs[e + 1]] - h @ w2).abs() <= bound * (1 + 1e-6)).all()


@pytest.mark.parametrize("x,w", [(-112, 90), (-122, 100), (-135, 115)])
def test_small_activations(x, w):
    """Activations of the order of 2^x against weights of the order of 2^w: ordinary sums."""
    def change(layer):
        layer["X"] = (layer["X"].double() * 2.0 ** x).float()
        for n in ("W1", "W3"):
            layer[n] = layer[n] * 2.0 ** w
    H, want, bound, _ = run_layer(100, 132, 24, change)
    assert ((H.double() - want).abs() <= bound).all()


@pytest.mark.parametrize("T", [9, 24, 40])
@pytest.mark.parametrize("where,value", [("W2", float("inf")), ("W2", float("nan")), ("W2", 3.4e38), ("Ws2", float("inf")),
                                         ("Ws2", float("nan")), ("Ws2", 3.4e38), ("X", 3.4e38)])
def test_values_that_are_not_finite(where, value, T):
    """A value in the second half's weights reaches its column alone, one in the activations its token's rows alone."""
    d, I, Is, k, n = 100, 68, 132, 40, 70
    w = synth.Workload("f32_values", T=T, d=d, E=2, I=I, K=2, K_base=1, budget=2 * T, dtype="f32", I_shared=Is,
                       I_shared_each=Is)

    def change(layer):
        if where == "X":
            layer["X"][T // 2, k] = value
        elif where == "W2":
            layer["W2"][0, k, n] = value
        else:
            layer["Ws2"][k, n] = value
    layer, H, O, offs, Hs, Os = second_half(w, change)
    if where == "X":   # (its scores stay finite, its sums do not)
        assert not torch.isfinite(Hs[T // 2]).all()
        others = torch.arange(T) != T // 2
        assert torch.isfinite(Hs[others]).all() and torch.isfinite(Os[others]).all()
        return
    for out, h, w2, rows, bad in ((O, H, layer["W2"][0], slice(offs[0], offs[1]), where == "W2"),
                                  (O, H, layer["W2"][1], slice(offs[1], offs[2]), False),
                                  (Os, Hs, layer["Ws2"], slice(0, T), where == "Ws2")):
        got, h = out[rows].double(), h[rows].double()
        want = (h @ w2.double()).float().double()
        mag = h.abs() @ w2.double().abs()
        finite = torch.isfinite(want)
        assert torch.equal(torch.isnan(got), torch.isnan(want))
        assert torch.equal(got[~finite & ~torch.isnan(want)], want[~finite & ~torch.isnan(want)])
        assert ((got - want).abs()[finite] <= (2 * Is * 2.0 ** -24 * mag)[finite]).all()
        assert finite.all() or (bad and finite[:, torch.arange(d) != n].all())
