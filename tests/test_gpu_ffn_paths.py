"""Every combination of kernels and streams that a bf16 layer's expert networks can take, each named
and asserted with the rule that chooses it: outputs against the oracle on a sample of tokens, and
outputs and intermediates bit for bit over repeated calls.  Protocol and tolerance of
tests/test_gpu_layer.py."""
import pytest
import torch

from paper_2604_08133_amd import synth
from paper_2604_08133_amd.layer import DeviceLayer
from tests.ffn_choice import choice_of
from tests.test_gpu_fp8 import quantised_reference
from tests.test_gpu_layer import check_layer, sample_tokens

pytestmark = pytest.mark.gpu

NAMES = {"streaming": (False, False, False), "tiled": (True, True, False),
         "beside: both tiled": (True, True, True), "beside: routed streaming": (False, True, True),
         "beside: shared streaming": (True, False, True),
         "shared tiled": (False, True, False)}


def check_path(w, path, layer, dev, ref=None):
    assert choice_of(w) == NAMES[path]
    check_layer(w, layer, dev=dev, ref_layer=ref, tokens=[0, w.T - 1, *sample_tokens(w.T, 6, 3)], tag=path)
    first = dict(dev.intermediates(), Y=dev.forward())
    torch.cuda.synchronize()
    first = {k: v.clone() for k, v in first.items()}
    for _ in range(3):
        again = dict(Y=dev.forward())
        torch.cuda.synchronize()
        again.update(dev.intermediates())
        for k, v in first.items():
            assert torch.equal(v.view(torch.uint8), again[k].view(torch.uint8)), k


SMALL = [  # path, T, d, E, I, I_shared, K, K_base, budget
    ("streaming", 300, 256, 8, 128, 128, 3, 1, 500),
    ("tiled", 700, 512, 16, 512, 512, 4, 1, 1600),
    ("tiled", 300, 512, 64, 128, 8192, 4, 0, 75),                      # by the shared expert alone
    ("beside: routed streaming", 330, 512, 16, 128, 16384, 4, 0, 40),
    ("beside: both tiled", 400, 512, 8, 512, 16384, 4, 0, 1280),
    ("tiled", 513, 1024, 6, 384, 0, 4, 0, 2052),
    ("streaming", 100, 512, 8, 128, 8192, 3, 1, 200),                  # few tokens, mostly shared expert
    ("tiled", 300, 1024, 1, 64, 4096, 1, 0, 0),                        # no routed pair
]


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("path,T,d,E,I,Is,K,Kb,budget", SMALL)
def test_smaller_layers(path, T, d, E, I, Is, K, Kb, budget, fp8):
    if fp8 and I % 128:
        pytest.skip("8-bit weights: widths are multiples of 128")
    w = synth.Workload("paths", T=T, d=d, E=E, I=I, K=K, K_base=Kb, budget=budget, dtype="bf16",
                       I_shared=Is, I_shared_each=Is, bias_kind="normal")
    layer = synth.make_layer(w, seed=91)
    ref = quantised_reference(layer)[0] if fp8 else None
    check_path(w, path, layer, DeviceLayer(w, layer, weights_fp8=fp8), ref)


@pytest.fixture(scope="module")
def large():
    """One layer above the size limit, and what its 8-bit codes stand for."""
    w = synth.deepseek_prefill(T=500, budget=1500)
    layer = {k: v.cpu() if v is not None else None
             for k, v in synth.make_layer(w, seed=92, device="cuda:0").items()}
    return w, layer, quantised_reference(layer)[0]


@pytest.mark.parametrize("fp8", [False, True])
def test_large_layer(large, fp8):
    w0, layer0, ref0 = large
    packed = None
    for path, T, budget in (("beside: both tiled", 500, 1500), ("beside: routed streaming", 200, 300),
                            ("beside: shared streaming", 100, 600), ("streaming", 60, 180)):
        w = w0.with_(T=T, budget=budget)
        layer, ref = dict(layer0, X=layer0["X"][:T].contiguous()), dict(ref0, X=ref0["X"][:T].contiguous())
        dev = packed = packed or DeviceLayer(w, layer, weights_fp8=fp8)
        dev.w, dev.X = w, layer["X"].cuda()
        check_path(w, path, layer, dev, ref if fp8 else None)


def test_large_layer_without_a_shared_expert_or_routed_pairs(large):
    w0, layer0, _ = large
    w = w0.with_(T=300, I_shared=0, I_shared_each=0, budget=900)
    layer = dict(layer0, X=layer0["X"][:300].contiguous(), Ws1=None, Ws3=None, Ws2=None)
    check_path(w, "tiled", layer, DeviceLayer(w, layer))
    w = w0.with_(T=200, budget=0, K_base=0)
    layer = dict(layer0, X=layer0["X"][:200].contiguous())
    check_path(w, "shared tiled", layer, DeviceLayer(w, layer))
