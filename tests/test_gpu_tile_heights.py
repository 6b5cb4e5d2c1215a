"""The bf16 tile kernel at every tile height (1 to 16 blocks of 16 rows, the last one partly
filled) and at contraction lengths that leave every remainder of its loop: one expert that
takes all tokens, so that the row count is the token count.  Same reference and tolerance as
tests/test_gpu_layer.py."""
import pytest

from paper_2604_08133_amd import synth
from paper_2604_08133_amd.layer import DeviceLayer
from tests.test_gpu_fp8 import quantised_reference
from tests.test_gpu_layer import check_layer, sample_tokens

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("d,I", [(256, 384), (768, 128), (512, 640)])
def test_every_tile_height(d, I, fp8):
    for blocks in range(1, 17):
        T = 16 * blocks - 3
        w = synth.Workload("one_expert", T=T, d=d, E=1, I=I, K=1, K_base=1, budget=T, dtype="bf16")
        layer = synth.make_layer(w, seed=70 + blocks)
        dev = DeviceLayer(w, layer, weights_fp8=fp8)
        ref = quantised_reference(layer)[0] if fp8 else None
        check_layer(w, layer, dev=dev, ref_layer=ref, tokens=sorted({0, T - 1, *sample_tokens(T, 12, blocks)}))


def test_light_tiles_among_full_ones():
    # strongly skewed experts: a few single tiles of at most 64 rows beside full tiles, at a
    # contraction length that is no multiple of the light tiles' longer weight ring
    w = synth.Workload("light_tiles", T=1500, d=512, E=10, I=640, K=2, K_base=1, budget=2600,
                       dtype="bf16", bias_kind="zipf")
    check_layer(w, synth.make_layer(w, seed=71), tokens=lambda offs, rt: sorted(
        {int(rt[r]) for e in range(10) for r in range(int(offs[e]), int(offs[e + 1])) if
         r - int(offs[e]) < 64}))
