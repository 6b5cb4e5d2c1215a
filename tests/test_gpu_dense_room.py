"""Tiled layers whose routed and shared experts share a launch: row tiles of the shared expert as
high as fit beside the routed workgroups in one round, and the usual ones where there is no room.
Protocol and tolerance of tests/test_gpu_layer.py."""
import pytest
import torch

from paper_2604_08133_amd import synth
from paper_2604_08133_amd.layer import DeviceLayer
from tests.ffn_choice import choice_of
from tests.test_gpu_fp8 import quantised_reference
from tests.test_gpu_layer import check_layer

pytestmark = pytest.mark.gpu


# expected routed workgroups of the first half (column tiles of 128 SwiGLU columns): 33, 210, 280,
# 210; the shared expert's 700 rows in tiles of 32, 192 (where the room is), 32, 192
@pytest.mark.parametrize("E,I,Is,fp8", [(8, 384, 640, False), (32, 704, 1216, False), (32, 1024, 640, False),
                                        (32, 768, 1280, True)])
def test_rows_beside_routed_tiles(E, I, Is, fp8):
    w = synth.Workload("room", T=700, d=512, E=E, I=I, K=4, K_base=1, budget=1600, dtype="bf16",
                       I_shared=Is, I_shared_each=Is, bias_kind="normal")
    assert choice_of(w) == (True, True, False)
    layer = synth.make_layer(w, seed=97)
    ref = quantised_reference(layer)[0] if fp8 else None
    check_layer(w, layer, dev=DeviceLayer(w, layer, weights_fp8=fp8), ref_layer=ref,
                tokens=[0, 31, 32, 191, 192, 383, 384, 575, 576, 699], tag="room")


# the shared expert beside routing and plan: less than a round of workgroups, a first round that
# leaves units free with a rest behind it, and more than two rounds (it starts after the routing);
# each call again right behind the first, on the same workspace, with equal results
@pytest.mark.parametrize("T,Is,fp8", [(300, 2816, False), (4096, 1408, False), (4096, 2816, False), (4096, 5632, False),
                                      (4096, 2816, True)])
def test_shared_expert_beside_routing(T, Is, fp8):
    w = synth.Workload("beside", T=T, d=2048, E=12, I=1408, K=4, K_base=1, budget=2 * T, dtype="bf16",
                       I_shared=Is, I_shared_each=Is, bias_kind="normal")
    w = w if T > 1000 else w.with_(E=48)
    assert choice_of(w) == (True, True, True)
    t = synth.make_layer(w, seed=98, device="cuda:0")
    dev = DeviceLayer(w, t, device="cuda:0", weights_fp8=fp8)
    Y = dev.forward().clone()
    for _ in range(3):
        again = dev.forward()
    assert torch.equal(Y, again)
    # the oracle's outputs on a few tokens
    layer = {k: v.cpu() if torch.is_tensor(v) else v for k, v in t.items()}
    ref = quantised_reference(layer)[0] if fp8 else None
    check_layer(w, layer, dev=dev, ref_layer=ref, tokens=[0, T // 3, T - 1], tag="beside")
