"""Weight-streaming kernel: contractions shorter than, as long as and longer than the loads a wave
has in flight, and the two widths of a workgroup in the second half with 8-bit weights (one column
block, two where there are more than 1024 of them).  Protocol and tolerance of
tests/test_gpu_layer.py."""
import pytest

from paper_2604_08133_amd import synth
from paper_2604_08133_amd.layer import DeviceLayer
from tests.ffn_choice import choice_of
from tests.test_gpu_fp8 import quantised_reference
from tests.test_gpu_layer import check_layer

pytestmark = pytest.mark.gpu


# a wave's steps: d / 64 and I / 64 (8 in flight), with 8-bit weights d / 128 and I / 128 (6, or 8
# where that is all of them; 12 in the second half with one column block)
@pytest.mark.parametrize("T,d,E,I,Is,budget,fp8", [
    (5, 64, 8, 64, 64, 9, False),
    (40, 512, 3, 512, 576, 70, False),
    (33, 576, 8, 1088, 0, 60, False),
    (5, 128, 8, 128, 128, 9, True),           # 4 x 10 workgroups
    (40, 768, 3, 896, 1536, 70, True),
    (33, 896, 8, 1664, 0, 60, True),
    (20, 2048, 24, 128, 768, 40, True),       # pairs of column blocks
    (24, 2048, 24, 896, 0, 48, True),
])
def test_contractions_and_widths(T, d, E, I, Is, budget, fp8):
    w = synth.Workload("stream", T=T, d=d, E=E, I=I, K=2, K_base=1, budget=budget, dtype="bf16",
                       I_shared=Is, I_shared_each=Is)
    assert choice_of(w) == (False, False, False)
    if fp8:   # workgroups of one column block: routed row tiles at most, then the shared expert's
        blocks = (min(E, budget) + (budget - min(E, budget)) // 32 + (-(-T // 32) if Is else 0)) * d // 32
        assert (blocks > 1024) == (d == 2048)
    layer = synth.make_layer(w, seed=95)
    ref = quantised_reference(layer)[0] if fp8 else None
    check_layer(w, layer, dev=DeviceLayer(w, layer, weights_fp8=fp8), ref_layer=ref, tag="stream")


# every length of the last pass and of the short rings: steps of a wave in the first and in the second
# half (bf16: rings of 4 and 8; 8-bit: of 2 and 4 up to four steps, of 4 and 8 up to eight (first half: seven and
# eight), else 3 and 6, second half 6 and 12)
@pytest.mark.parametrize("first,second,fp8", [
    (1, 16, False), (4, 9, False), (5, 10, False), (7, 11, False), (8, 12, False), (9, 13, False), (10, 14, False),
    (15, 3, False), (17, 24, False), (23, 25, False),
    (1, 3, True), (2, 4, True), (3, 1, True), (4, 2, True), (4, 4, True), (3, 7, True), (4, 9, True), (5, 10, True), (6, 12, True), (7, 13, True), (9, 17, True),
    (11, 23, True), (12, 25, True), (13, 6, True),
    (6, 5, True), (7, 8, True), (8, 3, True), (8, 6, True),
])
def test_steps_of_a_wave(first, second, fp8):
    step = 128 if fp8 else 64
    w = synth.Workload("steps", T=5, d=step * first, E=4, I=step * second, K=2, K_base=1, budget=9, dtype="bf16",
                       I_shared=step * first, I_shared_each=step * first)
    assert choice_of(w) == (False, False, False)
    layer = synth.make_layer(w, seed=96)
    ref = quantised_reference(layer)[0] if fp8 else None
    check_layer(w, layer, dev=DeviceLayer(w, layer, weights_fp8=fp8), ref_layer=ref, tag="steps")
