"""The work that a program using this library has it do, as cases that can be timed.

Three kinds of call, each through the C entry points (paper_2604_08133_amd.binding):

  layer   one forward pass of a budgeted MoE layer (allocmoe_moe_forward), weights packed
          when the model was loaded, workspace and output kept by the caller
  select  selection and dispatch from given scores, then the routing analytics
          (allocmoe_route_from_scores, allocmoe_dispatch, allocmoe_routing_stats)
  load    the re-tiling of one layer's weights when a model is loaded
          (allocmoe_pack_weights)

The shapes are those of the repository's workloads (synth.py, bench.py) or generic.
`listed` names the cases, `draw` gives others of the same ranges.
"""
import math
import statistics

import torch

from paper_2604_08133_amd import binding as B
from paper_2604_08133_amd import synth
from paper_2604_08133_amd.layer import DeviceLayer

DEVICE = "cuda:0"

# widths of the layer shapes: hidden, experts, expert width, shared width, width of one real
# shared expert, Top-K, gated shared expert
SHAPES = {
    "deepseek": dict(d=2048, E=64, I=1408, I_shared=2816, each=1408, K=6, gate=False),
    "qwen": dict(d=2048, E=60, I=1408, I_shared=5632, each=5632, K=4, gate=True),
    "olmoe": dict(d=2048, E=64, I=1024, I_shared=0, each=0, K=8, gate=False),
}
MAX_TOKENS = 16384


def layer_case(shape, T, budget, dtype="bf16", bias="none", fp8=False, selector="score", **widths):
    c = dict(kind="layer", T=T, budget=budget, K_base=1, dtype=dtype, bias=bias, fp8=fp8,
             selector=selector)
    c.update(SHAPES[shape] if shape else widths)
    return c


def listed():
    cases = {
        # one token of one request: latency, five short kernels in a chain
        "decode_1": layer_case("deepseek", 1, 3),
        # a decode batch at half budget: every active expert's weights once
        "decode_32": layer_case("deepseek", 32, 96),
        # a larger decode batch with 8-bit expert weights
        "decode_64_fp8": layer_case("deepseek", 64, 192, fp8=True),
        # a short ragged prompt, no shared expert, an odd budget
        "prompt_333_olmoe": layer_case("olmoe", 333, 1301),
        # a medium batch at three quarters of the budget, wide gated shared expert
        "prefill_2048_qwen": layer_case("qwen", 2048, 6144),
        # a prefill chunk with moderately skewed expert popularity
        "prefill_4096": layer_case("deepseek", 4096, 12288, bias="normal"),
        # a layer of the benchmark's stack: strong skew
        "stack_8192": layer_case("deepseek", 8192, 24576, bias="zipf"),
        # the longest batch: several requests' prompts in one call
        "prefill_16384": layer_case("deepseek", 16384, 49152, bias="zipf"),
        # a small model whose widths are multiples of 64 only, ragged token count
        "narrow_777": layer_case(None, 777, 1601, bias="normal", d=1088, E=32, I=704, I_shared=1408,
                                 each=704, K=4, gate=False),
        # full precision, as a model is checked or a small one is run; odd widths
        "fp32_500": layer_case(None, 500, 1000, dtype="f32", bias="normal", d=1000, E=16, I=700,
                               I_shared=1400, each=700, K=4, gate=True),
        # routing under study: selection, dispatch and analytics of given scores
        "select_6000": dict(kind="select", T=6000, E=64, K=6, K_base=1, budget=18001,
                            selector="score", levels=0),
        # loading a layer into the 8-bit format
        "load_fp8": dict(kind="load", d=2048, E=64, I=1408, I_shared=2816, fp8=True),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """Another case of the ranges above: token counts over their logarithm, any budget
    between a quarter and all of T*K, every weight format, selector and skew."""
    kind = rng.choice(["layer"] * 5 + ["narrow", "fp32", "select", "load"])
    bias = rng.choice(["none", "normal", "zipf"])
    ratio = rng.choice([0.25, 0.5, 0.75, 1.0, rng.uniform(0.25, 1.0)])

    def budget(T, K):
        return min(T * K, max(T, int(round(ratio * T * K))))

    if kind == "layer":
        limit = work(listed_case("prefill_16384"))["flops"]
        shape = rng.choice(["deepseek", "deepseek", "qwen", "olmoe"])
        T = _log_int(rng, 1, MAX_TOKENS)
        while True:
            c = layer_case(shape, T, budget(T, SHAPES[shape]["K"]), bias=bias, fp8=rng.random() < 0.25,
                           selector=rng.choice(["score"] * 4 + ["top_p", "relative"]))
            if work(c)["flops"] <= limit:
                return c
            T = T * 3 // 4
    if kind in ("narrow", "fp32"):
        K = rng.randint(2, 8)
        E = rng.randint(8, 64)
        shared = rng.choice([0, 1, 2])
        if kind == "narrow":
            d, I = 64 * rng.randint(4, 24), 64 * rng.randint(4, 24)
            T = _log_int(rng, 16, 4096)
        else:
            d, I = rng.randint(100, 1536), rng.randint(100, 1536)
            T = _log_int(rng, 16, 2048)
        return layer_case(None, T, budget(T, K), dtype="f32" if kind == "fp32" else "bf16", bias=bias,
                          d=d, E=E, I=I, I_shared=shared * I, each=I if shared else 0, K=K,
                          gate=bool(shared) and rng.random() < 0.5)
    if kind == "select":
        T, E = _log_int(rng, 16, MAX_TOKENS), rng.randint(16, 64)
        K = rng.randint(2, 8)
        return dict(kind="select", T=T, E=E, K=K, K_base=rng.randint(0, 1), budget=budget(T, K),
                    selector=rng.choice(["score", "top_p", "relative"]), levels=rng.choice([0, 0, 64]))
    step = rng.choice([64, 128])
    return dict(kind="load", d=step * rng.randint(512 // step, 2048 // step), E=rng.randint(8, 64),
                I=step * rng.randint(256 // step, 1408 // step), I_shared=step * rng.randint(0, 2816 // step),
                fp8=step == 128 and rng.random() < 0.7)


def listed_case(name):
    return next(c for c in listed() if c["name"] == name)


_SELECTORS = {"score": B.SELECT_SCORE, "top_p": B.SELECT_TOP_P, "relative": B.SELECT_RELATIVE}


def _workload(c):
    return synth.Workload("case", T=c["T"], d=c["d"], E=c["E"], I=c["I"], K=c["K"], K_base=c["K_base"],
                          budget=c["budget"], dtype=c["dtype"], I_shared=c["I_shared"],
                          I_shared_each=c["each"], shared_gate=c["gate"], bias_kind=c["bias"])


def prepare(case, seed):
    """What the program has before the call.  layer: activations, packed weights (row-major
    ones with fp32), workspace, output.  select: a batch's scores and the output arrays.
    load: the row-major weights and the buffer they go to."""
    c = case
    if c["kind"] == "layer":
        w = _workload(c)
        dev = DeviceLayer(w, synth.make_layer(w, seed=seed % 100003 + 1, device=DEVICE), device=DEVICE,
                          weights_fp8=c["fp8"])
        desc = dev.desc(selector=_SELECTORS[c["selector"]])
        return dict(kind="layer", desc=desc, dev=dev, ws=dev.workspace(desc),
                    Y=torch.empty((w.T, w.d), dtype=dev.dtype, device=DEVICE))
    if c["kind"] == "select":
        T, K = c["T"], c["K"]
        desc = B.make_desc(T, 64, c["E"], 64, K, c["K_base"], c["budget"], "f32",
                           selector=_SELECTORS[c["selector"]])
        ws_bytes = B.allocmoe_workspace_bytes(desc)
        i32 = dict(dtype=torch.int32, device=DEVICE)
        return dict(kind="select", desc=desc,
                    scores=synth.make_scores(T, c["E"], seed=seed % 100003 + 1,
                                             quantize_levels=c["levels"] or None).to(DEVICE),
                    topk_ids=torch.empty((T, K), **i32),
                    topk_s=torch.empty((T, K), dtype=torch.float32, device=DEVICE),
                    keep_count=torch.empty((T,), **i32), expert_offsets=torch.empty((c["E"] + 1,), **i32),
                    row_token=torch.empty((c["budget"],), **i32), row_rank=torch.empty((c["budget"],), **i32),
                    inv_row=torch.empty((T, K), **i32),
                    ws=torch.empty(ws_bytes, dtype=torch.uint8, device=DEVICE))
    w = synth.Workload("case", T=1, d=c["d"], E=c["E"], I=c["I"], K=1, K_base=1, budget=1, dtype="bf16",
                       I_shared=c["I_shared"], I_shared_each=c["I_shared"])
    t = synth.make_layer(w, seed=seed % 100003 + 1, device=DEVICE)
    desc = B.make_desc(w.T, w.d, w.E, w.I, w.K, w.K_base, w.budget, w.dtype, w.I_shared,
                       weights_fp8=c["fp8"])
    canonical = B.make_weights(**{n: t[n] for n in ("Wg", "W1", "W3", "W2", "Ws1", "Ws3", "Ws2")})
    # (zeros: the alignment gaps between the buffer's regions are never written)
    packed = torch.zeros(B.allocmoe_packed_bytes(desc), dtype=torch.uint8, device=DEVICE)
    return dict(kind="load", desc=desc, tensors=t, canonical=canonical, packed=packed)


def run(state):
    s = state
    if s["kind"] == "layer":
        B.allocmoe_moe_forward(s["desc"], s["dev"].X, s["dev"].weights, s["Y"], s["ws"])
        return s["Y"]
    if s["kind"] == "select":
        d = s["desc"]
        B.allocmoe_route_from_scores(d, s["scores"], s["topk_ids"], s["topk_s"], s["keep_count"], s["ws"])
        B.allocmoe_dispatch(d, s["topk_ids"], s["keep_count"], s["expert_offsets"], s["row_token"],
                            s["row_rank"], s["inv_row"], s["ws"])
        stats = B.allocmoe_routing_stats(d, s["scores"], s["topk_ids"], s["topk_s"], s["keep_count"])
        return dict(stats, **{n: s[n] for n in ("topk_ids", "topk_s", "keep_count", "expert_offsets",
                                                "row_token", "row_rank", "inv_row")})
    B.allocmoe_pack_weights(s["desc"], s["canonical"], s["packed"])
    return s["packed"]


def _active(E, pairs, bias):
    """Expected number of experts that `pairs` independent draws hit: experts alike, or with
    probabilities in proportion to exp of the gate's popularity bias (synth.make_layer)."""
    if bias == "zipf":
        p = [(i + 1) ** -1.1 for i in range(E)]
    elif bias == "normal":
        nd = statistics.NormalDist(0.0, math.sqrt(0.5))
        p = [math.exp(nd.inv_cdf((i + 0.5) / E)) for i in range(E)]
    else:
        p = [1.0] * E
    total = sum(p)
    return sum(1.0 - (1.0 - v / total) ** pairs for v in p)


def work(case):
    """Every input once, every output once; the layer's matrix products over the budgeted
    pairs and the shared expert.  Of the routed experts, those are expected to be read that
    the budgeted pairs hit when drawn with the popularity bias (see _active)."""
    c = case
    if c["kind"] == "select":
        T, K, E = c["T"], c["K"], c["E"]
        out = T * K * 12 + T * 8 + 8 * c["budget"] + E * 20
        return dict(bytes=T * E * 4 + out, flops=2 * T * E)
    d, E, I, Is = c["d"], c["E"], c["I"], c["I_shared"]
    if c["kind"] == "load":
        elems = 3 * d * (E * I + Is)
        return dict(bytes=elems * (3 if c["fp8"] else 4) + 2 * 2 * d * E, flops=elems if c["fp8"] else 0)
    T, Bn = c["T"], c["budget"]
    es = 4 if c["dtype"] == "f32" else 2
    active = _active(E, Bn, c["bias"])
    weights = 3 * d * (active * I + Is) * (1 if c["fp8"] else es)
    return dict(bytes=int(weights + d * E * es + 2 * T * d * es),
                flops=6 * d * (Bn * I + T * Is) + 2 * T * d * E)


def tolerance(case):
    c = case
    if c["kind"] == "load":
        return "exact"
    if c["kind"] == "select":
        return {"rel": 1e-5, "differ": 0.0}   # integers exact; fp32 sums of the analytics
    if c["dtype"] == "f32":
        # against the same layer in 64 bits: 1.1e-6, largest 8e-6
        return {"rel": 5e-6, "max": 1e-3}
    # Three roundings to bf16 on the way (H, O, Y): against the same layer in 64 bits 2.9e-3,
    # largest 1.6e-2.  `max` leaves room for a pair that ties with the selection's threshold
    # to within fp32 rounding: the two sides may keep another one of them.
    return {"rel": 1e-2, "max": 0.5}
