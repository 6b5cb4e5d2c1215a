"""Work that is more than one launch can hold (2^32 threads): nothing is left undone.  Inputs are
shared or repeated where that saves memory; results are checked where a short launch would end."""
import gc

import pytest
import torch

from paper_2604_08133_amd import binding as B
from paper_2604_08133_amd import synth
from paper_2604_08133_amd.layer import DeviceLayer

pytestmark = pytest.mark.gpu


def need(gigabytes):
    gc.collect()
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gigabytes * 1e9:
        pytest.skip(f"needs {gigabytes} GB of device memory")


def test_bf16_packing_of_a_very_large_layer():
    # 3.87e10 weights, 8 per thread; the matrices in between fit a launch each
    need(115)
    E, d, I = 64, 12288, 16384
    W = torch.empty(E * d * I, dtype=torch.int16, device="cuda").random_()
    Wg = torch.zeros((d, E), dtype=torch.bfloat16, device="cuda")
    desc = B.make_desc(1, d, E, I, 1, 1, 1, "bf16")
    packed = torch.zeros(B.allocmoe_packed_bytes(desc), dtype=torch.uint8, device="cuda")
    B.allocmoe_pack_weights(desc, B.make_weights(Wg=Wg, W1=W, W3=W, W2=W), packed)

    def fragments(e, Kd, N):   # [N/32][Kd/16] fragments of 64 lanes x 8 values
        m = W[e * d * I:(e + 1) * d * I].view(Kd // 16, 2, 8, N // 32, 32)
        return m.permute(3, 0, 1, 4, 2).reshape(N // 32, -1)

    out = packed[:E * 3 * d * I * 2].view(torch.int16)
    first, second = out[:E * 2 * d * I].view(E, I // 32, 2, -1), out[E * 2 * d * I:].view(E, d // 32, -1)
    for e in (0, 31, E - 1):
        want = fragments(e, d, I)
        assert torch.equal(first[e, :, 0], want) and torch.equal(first[e, :, 1], want)
        assert torch.equal(second[e], fragments(e, I, d))


def test_8bit_packing_of_a_very_wide_layer():
    # 8.39e6 strips of 32 columns, 512 threads each, in two launches: every expert as it is packed alone
    need(95)
    E, d, I = 64, 128, 2 ** 21 + 128
    W = torch.empty(E * d * I, dtype=torch.int16, device="cuda").random_()
    Wg = torch.zeros((d, E), dtype=torch.bfloat16, device="cuda")

    def pack(W, E):
        desc = B.make_desc(1, d, E, I, 1, 1, 1, "bf16", weights_fp8=True)
        packed = torch.zeros(B.allocmoe_packed_bytes(desc), dtype=torch.uint8, device="cuda")
        B.allocmoe_pack_weights(desc, B.make_weights(Wg=Wg, W1=W, W3=W, W2=W), packed)
        at13, at2 = 0, E * 2 * d * I
        scales13 = at2 + E * d * I + (5 * 16 * d * 2)
        scales2 = scales13 + (E * 2 * I * 4)
        return [packed[at13:at2].view(E, -1), packed[at2:at2 + E * d * I].view(E, -1),
                packed[scales13:scales2].view(E, -1), packed[scales2:scales2 + E * d * 4].view(E, -1)]

    whole = pack(W, E)
    for e in (0, 40, 63):
        for got, want in zip(whole, pack(W[e * d * I:(e + 1) * d * I], 1)):
            assert torch.equal(got[e], want[0])


def test_fp32_networks_of_a_very_large_batch():
    # 2^23 workgroups of routed rows and as many of the shared expert's in each first half
    need(160)
    w = synth.Workload("large_f32", T=2 ** 20, d=64, E=2, I=16384, K=1, K_base=1, budget=2 ** 20, dtype="f32",
                       I_shared=16384, I_shared_each=16384)
    t = synth.make_layer(w, seed=95, device="cuda:0")
    dev = DeviceLayer(w, t)
    dev.workspace(dev.desc()).zero_()
    Y = dev.forward()
    ids = dev.intermediates()["topk_ids"][:, 0].long()
    s = dev.intermediates()["topk_s"]
    rows = torch.cat([torch.arange(0, w.T, 5003, device="cuda"), torch.arange(w.T - 40, w.T, device="cuda")])
    x = t["X"][rows].double()
    net = lambda a, b, c: (torch.nn.functional.silu(x @ a.double()) * (x @ b.double())) @ c.double()
    routed = torch.stack([net(t["W1"][e], t["W3"][e], t["W2"][e]) for e in range(w.E)], dim=1)
    want = routed[torch.arange(len(rows), device="cuda"), ids[rows]] * s[rows].double() + net(t["Ws1"], t["Ws3"], t["Ws2"])
    assert float((Y[rows].double() - want).abs().max() / want.abs().max()) <= 1e-4
