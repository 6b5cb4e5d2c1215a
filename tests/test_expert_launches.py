"""Number of launches of the expert networks: the library's query against the launch structure counted by
hand, and the benchmark's record, which takes it from there."""
import ctypes

import pytest

import bench
from paper_2604_08133_amd import binding as B, synth


def deepseek(T, Bn, **kw):
    return B.make_desc(T, 2048, 64, 1408, 6, 0, Bn, "bf16", **{"I_shared": 2816, **kw})


@pytest.mark.parametrize("desc,launches", [
    (deepseek(32, 96), 2),                        # streaming, both groups in one launch a half
    (deepseek(100, 600), 4),                      # routed tiled beside a streaming shared expert
    (deepseek(130, 390), 4),                      # 14 workgroups a die: less than a round
    (deepseek(2048, 6144), 4),                    # 24
    (deepseek(4096, 12288), 5),                   # 48: the first round and the rest
    (deepseek(4096, 12288, weights_fp8=True), 5),
    (deepseek(8192, 24576), 4),                   # 88: the fork stands behind the routing kernel
    (deepseek(2048, 6144, I_shared=0), 2),
    (deepseek(2048, 0), 2),                       # no routed pairs
    (deepseek(2048, 0, I_shared=0), 0),
    (B.make_desc(2048, 2048, 60, 1408, 4, 1, 4096, "bf16", 5632, True), 5),
    (B.make_desc(777, 1088, 32, 704, 4, 1, 1601, "bf16", 1408), 2),   # one launch a half for both groups
])
def test_launches(desc, launches):
    assert B.allocmoe_expert_launches(desc) == launches


def test_bf16_only():
    n = ctypes.c_int32(-1)
    desc = B.make_desc(64, 128, 8, 256, 2, 1, 64, "f32")
    assert B.load().allocmoe_expert_launches(ctypes.byref(desc), ctypes.byref(n)) == B.EINVAL
    assert B.load().allocmoe_expert_launches(ctypes.byref(deepseek(32, 96)), None) == B.EINVAL
    assert n.value == -1


def test_benchmark_record():
    # 3 layers of 4096 tokens, one of them without routed pairs
    descs = [deepseek(4096, 12288), deepseek(4096, 12288), deepseek(4096, 0)]
    run = object.__new__(bench.Bench)
    run.B, run.name, run.fp8, run.w, run.descs = B, "prefill", True, synth.deepseek_stack_layer(12288, T=4096), descs
    run.devs = [None] * len(descs)
    roof, _ = run.analyse(1.5, dict.fromkeys(B.STAGES, 0.1), 64 * 3, 24576, None)
    assert roof["launches_per_step"] == 5 + 5 + 2 and "the 2/5 launches of a layer" in roof["kernel"]
