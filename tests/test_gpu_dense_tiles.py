"""The shared expert alone on the tile kernel, with few workgroups and many: every weight ring that
its row tiles may get, contractions of every remainder of those rings, the last row tile short."""
import pytest
import torch

from paper_2604_08133_amd import binding as B
from paper_2604_08133_amd import synth
from paper_2604_08133_amd.layer import DeviceLayer

pytestmark = pytest.mark.gpu


# second half (d columns: few column tiles): tiles of 32 rows, 12 steps of weights, Is / 64 slots;
# first half: the rows per tile below, 8 steps from 65 to 128 rows, 12 up to 64, d / 64 slots
@pytest.mark.parametrize("T,d,Is", [(130, 1088, 8192),    # 96 and 34 rows
                                    (80, 1152, 8256),     # 80
                                    (100, 1216, 8320),    # 100
                                    (128, 1024, 8384),    # 128
                                    (111, 1088, 8448),    # 111
                                    (65, 1344, 8512),     # 65
                                    (128, 1152, 4096),    # 32, one round
                                    (190, 1088, 4160),    # 64, 64, 62
                                    (300, 1024, 16640)])  # 256 and 44: above one round, the short rings
def test_shared_expert(T, d, Is):
    w = synth.Workload("dense", T=T, d=d, E=1, I=64, K=1, K_base=0, budget=0, dtype="bf16",
                       I_shared=Is, I_shared_each=Is)
    t = synth.make_layer(w, seed=T + d, device="cuda:0")
    dev = DeviceLayer(w, t, device="cuda:0")
    Y = dev.forward().double()
    X, W1, W3, W2 = (t[n].double() for n in ("X", "Ws1", "Ws3", "Ws2"))
    a = X @ W1
    H = a * torch.sigmoid(a) * (X @ W3)
    want = H @ W2
    # H, O and Y are rounded to bf16, H to a relative 2^-9 at most, evenly spread (standard
    # deviation 2^-9 / sqrt 3): 7 standard deviations of its part in the sum, and 2^-9 of the value
    # for each of the other two
    bound = 7 * 2.0 ** -9 / 3 ** 0.5 * ((H * H) @ (W2 * W2)).sqrt() + 2.0 ** -8 * want.abs()
    assert ((Y - want).abs() <= bound).all()
    again = dev.forward().double()
    assert torch.equal(Y, again)
