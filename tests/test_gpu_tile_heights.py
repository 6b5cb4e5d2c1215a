"""The bf16 tile kernel at every tile height (1 to 16 blocks of 16 rows, the last one partly
filled), at contraction lengths that leave every remainder of its loops (odd numbers of 64-k
slots among them) and at widths that end inside a column tile; and a layer of ragged widths with a
gated shared expert on both kernels.  Same reference and tolerance as tests/test_gpu_layer.py."""
import pytest
import torch

from paper_2604_08133_amd import synth
from paper_2604_08133_amd.layer import DeviceLayer
from tests.ffn_choice import choice_of
from tests.test_gpu_fp8 import quantised_reference
from tests.test_gpu_layer import check_layer, sample_tokens, stratified_tokens

pytestmark = pytest.mark.gpu

T, E = 3000, 64
WIDTHS = [
    (256, 384, 128, False), (768, 128, 0, False), (512, 640, 384, False), (320, 192, 192, False),
    (64, 1088, 64, False), (1088, 64, 0, False), (448, 832, 320, False), (704, 448, 1408, False),
    (256, 384, 128, True), (384, 256, 384, True), (640, 128, 0, True), (768, 640, 128, True)]
HEIGHTS = {}    # seen at each width


@pytest.mark.parametrize("d,I,I_shared,fp8", WIDTHS)
def test_tile_heights_and_widths(d, I, I_shared, fp8):
    # a ramp of popularity: single tiles of a few rows up to experts of several full tiles
    # (3.3 GFLOP and more at 140 rows an expert: the tile kernel's side of the rule)
    w = synth.Workload("tile_heights", T=T, d=d, E=E, I=I, K=4, K_base=1, budget=3 * T, dtype="bf16",
                       I_shared=I_shared, I_shared_each=I_shared, bias_kind="normal")
    layer = synth.make_layer(w, seed=71)
    assert choice_of(w)[0]
    layer["bias"] = torch.linspace(-3.0, 1.0, E)
    dev = DeviceLayer(w, layer, weights_fp8=fp8)
    ref = quantised_reference(layer)[0] if fp8 else None
    heights = set()

    def tokens(offs, row_token):
        for e in range(E):
            n = int(offs[e + 1]) - int(offs[e])
            tiles = -(-n // 256)
            per = -(-n // max(tiles, 1))
            heights.update(-(-min(per, n - i * per) // 16) for i in range(tiles))
        return stratified_tokens(offs, row_token, T)

    check_layer(w, layer, dev=dev, ref_layer=ref, tokens=tokens)
    # (a height may be missing at one width)
    assert len(heights) >= 12 and min(heights) <= 2 and max(heights) == 16, heights
    HEIGHTS[d, I, I_shared, fp8] = heights


@pytest.mark.parametrize("fp8", [False, True])
def test_the_widths_together_leave_no_height_out(fp8):
    widths = [w for w in WIDTHS if w[3] == fp8]
    if any(w not in HEIGHTS for w in widths):
        pytest.skip("not all widths were run")
    assert set().union(*(HEIGHTS[w] for w in widths)) == set(range(1, 17))


@pytest.mark.parametrize("T,budget", [(32, 127), (40, 128), (128, 512), (500, 1000), (700, 2800)])
def test_both_sides_of_the_kernel_choice(T, budget):
    # 8 to 175 rows per expert, up to 1.7 GFLOP streaming, from 4.5 tiled (the limits of the rule
    # themselves: tests/test_ffn_choice.py)
    w = synth.Workload("choice", T=T, d=832, E=16, I=448, K=4, K_base=1, budget=budget, dtype="bf16",
                       I_shared=896, I_shared_each=448, shared_gate=True, bias_kind="normal")
    assert choice_of(w) == (T >= 500, T >= 500, False)
    check_layer(w, synth.make_layer(w, seed=73), tokens=[0, T - 1, *sample_tokens(T, 24, 9)])
