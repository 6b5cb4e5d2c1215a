"""Re-tiling of bf16 weights byte for byte: widths of whole and half 128-column strips, the
fewest k blocks, matrices that start at an odd element, both shared and no shared expert."""
import pytest
import torch

from paper_2604_08133_amd import binding as B, synth

pytestmark = pytest.mark.gpu


def fragments(W):
    """[G, Kd, N] -> [G, N/32, Kd/16, lane, 8]: lane 32 h + c holds k = 16 kb + 8 h + i, n = 32 nb + c."""
    G, Kd, N = W.shape
    f = W.view(torch.int16).reshape(G, Kd // 16, 2, 8, N // 32, 32)
    return f.permute(0, 4, 1, 2, 5, 3).reshape(G, N // 32, Kd // 16, 64, 8)


@pytest.mark.parametrize("d,I,I_shared,odd", [(64, 64, 0, False), (128, 64, 128, True), (64, 192, 64, False),
                                              (192, 320, 448, True), (1088, 128, 0, True),
                                              (256, 1024, 2048, False)])
def test_fragments(d, I, I_shared, odd):
    E = 3
    w = synth.Workload("pack_bf16", T=1, d=d, E=E, I=I, K=1, K_base=1, budget=1, dtype="bf16",
                       I_shared=I_shared, I_shared_each=I_shared)
    t = synth.make_layer(w, seed=83)
    names = ["W1", "W3", "W2"] + (["Ws1", "Ws3", "Ws2"] if I_shared else [])

    def device_copy(x):
        buf = torch.empty(x.numel() + 1, dtype=x.dtype, device="cuda")
        part = buf[1:] if odd else buf[:-1]
        return part.view(x.shape).copy_(x)

    dev = {n: device_copy(t[n]) for n in names}
    desc = B.make_desc(1, d, E, I, 1, 1, 1, "bf16", I_shared)
    packed = torch.zeros(B.allocmoe_packed_bytes(desc), dtype=torch.uint8, device="cuda")
    B.allocmoe_pack_weights(desc, B.make_weights(Wg=t["Wg"].cuda(), **dev), packed)
    got = packed.cpu().view(torch.int16)
    at = 0
    for n1, n3, n2 in (names[:3], names[3:]) if I_shared else (names,):
        f1, f3, f2 = (fragments(t[n].reshape(-1, *t[n].shape[-2:])) for n in (n1, n3, n2))
        for want in (torch.cat([f1.flatten(2), f3.flatten(2)], dim=2), f2):
            assert torch.equal(got[at:at + want.numel()], want.reshape(-1)), (n1, n2)
            at += want.numel()
