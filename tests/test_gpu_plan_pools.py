"""Selection and dispatch of the one-launch plan kernel where its paths change: pools that one wave
ranks directly, pools with one and with several entries a thread, ties at the threshold (few, and more
than a wave ranks), one and sixteen pool entries per token, the largest sizes of every block size (256,
512 and 1024 threads), candidate rows that do not fit the LDS, and the token count from which on
dispatch is a sequence of launches.  Bit for bit against the oracle run from the same scores."""
import pytest

from paper_2604_08133_amd import synth
from paper_2604_08133_amd.layer import DeviceLayer
from tests.test_gpu_layer import check_layer
from tests.test_gpu_route_dispatch import assert_same, gpu_route_dispatch, oracle_route_dispatch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,K,Kb,levels", [
    (1, 8, 2, 1, 0), (16, 16, 5, 1, 0), (13, 16, 5, 0, 0), (64, 64, 2, 1, 4),       # pools of 1, 64, 65, 64
    (85, 20, 4, 1, 0), (64, 20, 5, 1, 0), (64, 20, 5, 1, 3), (256, 20, 2, 1, 0),     # 255, 256: an entry a thread
    (86, 20, 4, 1, 0), (86, 20, 4, 1, 2),                                          # 258: a second entry for some
    (333, 64, 8, 1, 0), (333, 64, 8, 1, 64), (1000, 64, 6, 0, 3),
    (256, 64, 16, 0, 0), (256, 64, 16, 0, 64), (257, 64, 16, 0, 0), (257, 64, 16, 0, 64),   # 256, 512 threads
    (512, 64, 16, 0, 0), (512, 64, 16, 0, 64), (513, 64, 16, 0, 0), (513, 64, 16, 0, 64),   # 512, 1024 threads
    (768, 33, 16, 0, 0), (1024, 40, 12, 0, 256),                                   # 12 entries a thread
    (1024, 64, 16, 15, 0), (1025, 64, 6, 1, 0), (3000, 64, 16, 0, 16),
    (6143, 64, 6, 1, 0), (6144, 64, 6, 1, 0),                                      # dispatch: one launch, a sequence
    (3072, 64, 16, 0, 0),                                                          # 48 a thread, all ids in LDS
    (3500, 64, 15, 3, 0), (8192, 64, 7, 1, 64),                                    # ids read where they are used
])
def test_selection_and_dispatch(T, E, K, Kb, levels):
    scores = synth.make_scores(T, E, seed=31, quantize_levels=levels or None)
    n_pool = T * (K - Kb)
    for extra in sorted({0, 1, n_pool // 3, n_pool // 2 + 1, n_pool - 1, n_pool}):
        args = (scores, K, Kb, T * Kb + extra)
        # (without a workspace one workgroup selects whatever the size)
        assert_same(gpu_route_dispatch(*args, select_ws=False), oracle_route_dispatch(*args), extra)


@pytest.mark.parametrize("T,K,Kb,distinct", [(40, 4, 1, 40), (300, 4, 1, 3), (700, 6, 0, 2), (1500, 4, 1, 5),
                                             (6143, 4, 1, 6143), (6143, 4, 1, 9), (6144, 4, 1, 6144), (6144, 4, 1, 9)])
def test_one_launch_for_both(T, K, Kb, distinct):
    # repeated tokens: equal scores at the threshold, some of them kept
    for budget in (T * Kb + 1, T * Kb + T // 2, T * K - 3):
        w = synth.Workload("plan", T=T, d=128, E=16, I=64, K=K, K_base=Kb, budget=budget, dtype="bf16", I_shared=0)
        layer = synth.make_layer(w, seed=32)
        layer["X"] = layer["X"][:distinct].repeat(-(-T // distinct), 1)[:T].contiguous()
        check_layer(w, layer, dev=DeviceLayer(w, layer), tokens=[0, T // 2, T - 1], tag="plan")
