"""Packing of 8-bit expert weights where its kernel can go wrong: columns shorter and longer
than the 2048 rows that stay in registers, the last column strip, scales outside the range of
the short division, zeros of either sign.  Codes and scales byte for byte against the
oracle's quantiser."""
import numpy as np
import pytest
import torch

from oracle import quant
from paper_2604_08133_amd import binding as B, synth
from tests.test_gpu_fp8 import align256, fragments

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,I,values", [(128, 128, "normal"), (2048, 384, "normal"), (2176, 128, "normal"),
                                        (256, 128, "columns"), (256, 256, "exact")])
def test_codes_and_scales(d, I, values):
    w = synth.Workload("pack_fp8", T=1, d=d, E=2, I=I, K=1, K_base=1, budget=1, dtype="bf16")
    t = synth.make_layer(w, seed=81, only=("Wg", "W1", "W3", "W2"))
    g = torch.Generator().manual_seed(82)
    if values == "columns":      # scales from the smallest to near the largest exponent
        for n in ("W1", "W3", "W2"):
            e = torch.randint(-125, 110, (t[n].shape[-1],), generator=g).float()
            t[n] = (t[n].float() * torch.exp2(e)).bfloat16()
    elif values == "exact":      # quotients on the rounding boundaries, zeros of both signs
        for n in ("W1", "W3", "W2"):
            t[n] = torch.randint(-28, 29, t[n].shape, generator=g).bfloat16()
            t[n][0, :, 0] = 0.0
            t[n][1, :, -1] = -0.0
    desc = B.make_desc(1, d, 2, I, 1, 1, 1, "bf16", weights_fp8=True)
    dev = {n: t[n].cuda() for n in ("Wg", "W1", "W3", "W2")}
    packed = torch.zeros(B.allocmoe_packed_bytes(desc), dtype=torch.uint8, device="cuda")
    B.allocmoe_pack_weights(desc, B.make_weights(**dev), packed)
    got = packed.cpu().numpy()
    q = {n: quant.quantise_columns(t[n].float().numpy()) for n in ("W1", "W3", "W2")}
    want13 = np.concatenate([fragments(q["W1"][0]), fragments(q["W3"][0])], axis=2).reshape(-1)
    want2 = fragments(q["W2"][0]).reshape(-1)
    at2 = align256(want13.size)
    at_gate = at2 + align256(want2.size)
    at_s13 = at_gate + align256(5 * 16 * d * 2)
    at_s2 = at_s13 + align256(2 * 2 * I * 4)
    assert np.array_equal(got[:want13.size], want13)
    assert np.array_equal(got[at2:at2 + want2.size], want2)
    assert np.array_equal(got[at_s13:at_s13 + 2 * 2 * I * 4].view(np.float32).reshape(2, 2, I),
                          np.stack([q["W1"][1], q["W3"][1]], axis=1))
    assert np.array_equal(got[at_s2:at_s2 + 2 * d * 4].view(np.float32).reshape(2, d), q["W2"][1])
