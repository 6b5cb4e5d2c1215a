"""The library's one extra stream and its events under several callers: host threads with a stream each,
whose layers fork before and behind the routing kernel, and one thread that enqueues on two streams in
turn.  Every output is the one that the layer gives alone."""
import threading

import pytest
import torch

from paper_2604_08133_amd import binding as B, synth
from paper_2604_08133_amd.layer import DeviceLayer
from tests.ffn_choice import choice_of

pytestmark = pytest.mark.gpu


class Caller:
    def __init__(self, T, Is, seed):
        w = synth.Workload("caller", T=T, d=1024, E=8, I=256, K=2, K_base=1, budget=3 * T // 2, dtype="bf16",
                           I_shared=Is, I_shared_each=Is, bias_kind="normal")
        assert choice_of(w) == (True, True, True)
        self.dev = DeviceLayer(w, synth.make_layer(w, seed=seed, device="cuda:0"))
        self.desc = self.dev.desc()
        self.ws = self.dev.workspace(self.desc)
        self.want = self.dev.forward().clone()
        self.out = [torch.empty_like(self.want) for _ in range(6)]
        torch.cuda.synchronize()
        self.stream = torch.cuda.Stream()

    def enqueue(self, Y):
        B.allocmoe_moe_forward(self.desc, self.dev.X, self.dev.weights, Y, self.ws, self.stream)

    def check(self):
        for Y in self.out:
            assert torch.equal(Y, self.want)


def callers():
    # 48 workgroups a die (fork before routing, two launches), 24 (one launch), 96 (fork behind routing)
    made = [Caller(4096, 2816, 101), Caller(2048, 2816, 102), Caller(8192, 2816, 103)]
    assert [B.allocmoe_expert_launches(c.desc) for c in made] == [5, 4, 4]
    return made


def test_one_thread_several_streams():
    cs = callers()
    for i in range(6):
        for c in cs:
            c.enqueue(c.out[i])
    torch.cuda.synchronize()
    for c in cs:
        c.check()


def test_threads_with_a_stream_each():
    cs = callers()
    errors = []

    def work(c):
        try:
            for Y in c.out:
                c.enqueue(Y)
        except Exception as e:   # (reported by the test's own thread)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(c,)) for c in cs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors
    for c in cs:
        c.check()
