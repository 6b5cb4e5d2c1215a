"""The fp32 tile kernel at its edges: contraction depths with every remainder of a 16-k step
and fewer steps than waves, column counts with every remainder of a lane's 4 columns, rows
around one and two 16-row blocks, widths below 4 (the one-thread-per-output kernel), and the
two kernels side by side in one layer.  Same reference and tolerance as
tests/test_gpu_layer.py (fp32: sums of at most 300 products in another order, 1e-4)."""
import pytest

from paper_2604_08133_amd import synth
from tests.test_gpu_layer import check_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,I,Ish", [(4, 4, 4), (5, 7, 6), (16, 64, 65), (17, 63, 66), (66, 67, 129),
                                     (131, 34, 35), (300, 133, 70), (1, 5, 3), (3, 2, 1), (9, 3, 40),
                                     (40, 9, 2), (128, 16, 0)])
@pytest.mark.parametrize("T", [1, 15, 16, 17, 33, 70])
def test_widths_and_rows(d, I, Ish, T):
    w = synth.Workload("f32_tiles", T=T, d=d, E=3, I=I, K=2, K_base=1, budget=T + T // 2, dtype="f32",
                       I_shared=Ish, I_shared_each=Ish, shared_gate=bool(Ish) and T % 2 == 1,
                       bias_kind="normal")
    check_layer(w, synth.make_layer(w, seed=90 + T))
