"""Packing of 8-bit expert weights where its kernel can go wrong: columns shorter and longer
than the 2048 rows that stay in registers, the last column strip, scales outside the range of
the short division, zeros of either sign, NaNs and infinities.  Codes and scales byte for byte against the
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


def test_nan_and_infinite_weights():
    # A NaN takes the largest code with its own sign and leaves the rest of its column as it is
    # without it (scale 1 where nothing else is left); an infinity makes the scale infinite.
    d, I, E = 2176, 128, 2      # columns of W1 and W3 in two chunks of rows, those of W2 in one
    w = synth.Workload("pack_fp8", T=1, d=d, E=E, I=I, K=1, K_base=1, budget=1, dtype="bf16")
    t = synth.make_layer(w, seed=83, only=("Wg", "W1", "W3", "W2"))
    q, codes = {}, {}
    for n in ("W1", "W3", "W2"):
        bits = t[n].view(torch.int16)
        last = bits.shape[1] - 1
        nan = torch.zeros(bits.shape, dtype=torch.bool)
        for pattern, at in ((0x7FC0, (0, 7, 3)), (0xFFC1, (0, last, 4)), (0x7F81, (1, 40, 5)), (0xFFFF, (1, 0, 6)),
                            (0x7FC0, (0, slice(None), 9)), (0xFFC0, (1, 33, 10))):
            bits[at] = pattern - (1 << 16 if pattern >> 15 else 0)
            nan[at] = True
        t[n][1, :, 10] = torch.where(nan[1, :, 10], t[n][1, :, 10], 0.0)    # one NaN among zeros
        t[n][0, 5, 11] = float("inf")
        t[n][1, 6, 12] = -float("inf")
        values = t[n].float().masked_fill(nan, 0.0).numpy()
        inf = np.isinf(values)
        c, s = quant.quantise_columns(np.where(inf, 0.0, values))
        column = inf.any(axis=1, keepdims=True)
        s = np.where(column[:, 0], np.float32(np.inf), s)
        c = np.where(column, np.where(np.signbit(values), 0x80, 0), c)
        # (infinity over infinity: the largest code, of no particular sign)
        codes[n] = np.where(nan.numpy(), np.where(bits.numpy() < 0, 0xFE, 0x7E), c).astype(np.uint8), inf
        q[n] = s.astype(np.float32)
    desc = B.make_desc(1, d, E, I, 1, 1, 1, "bf16", weights_fp8=True)
    packed = torch.zeros(B.allocmoe_packed_bytes(desc), dtype=torch.uint8, device="cuda")
    B.allocmoe_pack_weights(desc, B.make_weights(**{n: t[n].cuda() for n in ("Wg", "W1", "W3", "W2")}), packed)
    got = packed.cpu().numpy()
    sides = [np.concatenate([fragments(codes["W1"][i].astype(np.uint8)), fragments(codes["W3"][i].astype(np.uint8))],
                            axis=2).reshape(-1) for i in (0, 1)]
    second = [fragments(codes["W2"][i].astype(np.uint8)).reshape(-1) for i in (0, 1)]
    at2 = align256(sides[0].size)
    for at, (want, inf) in ((0, sides), (at2, second)):
        part = got[at:at + want.size]
        assert np.array_equal(part[inf == 0], want[inf == 0])
        assert (part[inf == 1] & 0x7F == 0x7E).all() and inf.sum() > 0
    at_s13 = at2 + align256(second[0].size) + align256(5 * 16 * d * 2)
    at_s2 = at_s13 + align256(E * 2 * I * 4)
    assert np.array_equal(got[at_s13:at_s13 + E * 2 * I * 4].view(np.float32).reshape(E, 2, I),
                          np.stack([q["W1"], q["W3"]], axis=1))
    assert np.array_equal(got[at_s2:at_s2 + E * d * 4].view(np.float32).reshape(E, d), q["W2"])
