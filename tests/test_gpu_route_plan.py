"""Layers of up to 16 tokens, whose routing workgroup selects and dispatches as well: pools from one entry
to 256, every budget that the pool's ends and middle give, equal tokens (ties at the threshold), up to 16
candidates, few and 64 experts, and the selectors; and 17 tokens, which take two launches.  Indices bit
for bit against the oracle from the same scores, outputs as in tests/test_gpu_layer.py."""
import pytest
import torch

import oracle
from paper_2604_08133_amd import binding as B, synth
from paper_2604_08133_amd.layer import DeviceLayer
from tests.test_gpu_fp8 import quantised_reference
from tests.test_gpu_layer import check_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,K,Kb,distinct", [(1, 2, 2, 1, 1), (1, 64, 16, 0, 1), (2, 64, 6, 1, 1), (7, 9, 9, 2, 7),
                                               (15, 64, 6, 1, 4), (16, 64, 16, 0, 16), (16, 20, 16, 0, 2),
                                               (16, 5, 4, 3, 16), (16, 16, 3, 3, 16), (17, 64, 16, 0, 3)])
def test_budgets(T, E, K, Kb, distinct):
    n_pool = T * (K - Kb)
    for extra in sorted({0, min(1, n_pool), n_pool // 2, max(0, n_pool - 1), n_pool}):
        w = synth.Workload("route_plan", T=T, d=192, E=E, I=64, K=K, K_base=Kb, budget=T * Kb + extra, dtype="bf16",
                           I_shared=64 * (T % 2), I_shared_each=64, shared_gate=T == 15, bias_kind="normal")
        layer = synth.make_layer(w, seed=5 + T)
        layer["X"] = layer["X"][:distinct].repeat(-(-T // distinct), 1)[:T].contiguous()
        check_layer(w, layer, dev=DeviceLayer(w, layer), tag="route_plan")


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("T,K,budget", [(1, 6, 3), (16, 16, 100), (16, 6, 17), (11, 5, 40)])
def test_selectors(mode, T, K, budget):
    w = synth.Workload("route_plan", T=T, d=128, E=33, I=64, K=K, K_base=1, budget=budget, dtype="bf16", I_shared=0,
                       I_shared_each=0, bias_kind="normal")
    dev = DeviceLayer(w, synth.make_layer(w))
    desc = dev.desc(selector=mode)
    ws = dev.workspace(desc)
    Y = torch.empty((T, w.d), dtype=torch.bfloat16, device="cuda:0")
    print(f"selector {mode} T={T} K={K} B={budget}", flush=True)
    B.allocmoe_moe_forward(desc, dev.X, dev.weights, Y, ws)
    torch.cuda.synchronize()
    L = B.allocmoe_workspace_layout(desc)
    got = lambda at, shape, dtype=torch.int32: B.ws_view(ws, at, shape, dtype).cpu()
    from oracle import selectors as sel
    ids, s = oracle.topk(got(L.scores, (T, w.E), torch.float32), K)
    kept, keep = sel.select(s, mode, 1, budget)
    offs, row_token, row_rank, inv = oracle.dispatch(ids, kept, w.E)
    assert torch.equal(got(L.topk_ids, (T, K)), ids) and torch.equal(got(L.topk_s, (T, K), torch.float32), s)
    assert torch.equal(got(L.sel_keys, (T, K), torch.float32), torch.from_numpy(sel.selector_keys(s, mode)))
    assert torch.equal(got(L.keep_count, (T,)), keep) and torch.equal(got(L.expert_offsets, (w.E + 1,)), offs)
    assert torch.equal(got(L.row_token, (budget,)), row_token) and torch.equal(got(L.row_rank, (budget,)), row_rank)
    assert torch.equal(got(L.inv_row, (T, K)), inv)


# the shared expert's first half in the routing launch: one step a wave and uneven numbers of steps, below and
# above its ring of four (8-bit weights three); the widest shared expert that takes one round and the first that does not; d too short
@pytest.mark.parametrize("T,d,Is,gate,fp8", [(1, 256, 64, False, False), (16, 320, 128, True, False), (5, 192, 64, False, False),
                                             (3, 1088, 192, False, False), (9, 1216, 64, True, False), (16, 2048, 64, False, False),
                                             (2, 256, 8128, False, False), (2, 256, 8192, False, False),
                                             (1, 512, 128, False, True), (16, 640, 256, True, True), (7, 384, 128, False, True),
                                             (4, 2048, 128, False, True), (11, 2432, 128, False, True)])
def test_shared_expert_beside(T, d, Is, gate, fp8):
    w = synth.Workload("route_shared", T=T, d=d, E=6, I=128, K=3, K_base=1, budget=2 * T, dtype="bf16", I_shared=Is,
                       I_shared_each=Is, shared_gate=gate)
    layer = synth.make_layer(w, seed=11)
    ref = quantised_reference(layer)[0] if fp8 else None
    check_layer(w, layer, dev=DeviceLayer(w, layer, weights_fp8=fp8), ref_layer=ref, tag="beside")
