"""Tiled layers whose routed and shared experts share a launch: row tiles of the shared expert as
high as fit beside the routed workgroups in one round, and the usual ones where there is no room.
Protocol and tolerance of tests/test_gpu_layer.py."""
import pytest

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
