"""The rule that chooses kernel and stream of the bf16 expert networks (csrc/choice.hpp), compiled
from its header by the host compiler, for tests that name the path they take."""
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_08133_amd", "csrc")
SOURCE = """
#include "choice.hpp"
extern "C" int choose(int T, int d, int E, int I, int Is, long long B) {
    const allocmoe::FfnChoice c = allocmoe::choose_ffn(T, d, E, I, Is, B);
    return c.routed_tiled | c.shared_tiled << 1 | c.own_stream << 2;
}
extern "C" int second_half(int T, int d, int E, int I, int Is, long long B, int weight_bytes) {
    return allocmoe::side_second_half_workgroups(T, d, E, I, Is, B, weight_bytes);
}
extern "C" int beside_route(int T, int d, int E, int I, int Is, long long B, int fp8) {
    return allocmoe::first_half_beside_route(allocmoe::choose_ffn(T, d, E, I, Is, B), T, d, Is, B, fp8);
}
extern "C" int tile_rows(long long rows, int col_tiles, long long most) {
    return allocmoe::dense_tile_rows(rows, col_tiles, most);
}
"""


@functools.lru_cache(maxsize=None)
def _library():
    with tempfile.TemporaryDirectory() as tmp:
        src, lib = os.path.join(tmp, "choose.cpp"), os.path.join(tmp, "choose.so")
        with open(src, "w") as f:
            f.write(SOURCE)
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                               src, "-o", lib])
        return ctypes.CDLL(lib)


def choose(T, d, E, I, Is, B):
    """(routed experts on the tile kernel, shared expert on the tile kernel, shared expert on the
    library's own stream)"""
    bits = _library().choose(T, d, E, I, Is, ctypes.c_longlong(B))
    return bool(bits & 1), bool(bits & 2), bool(bits & 4)


def second_half_workgroups(T, d, E, I, Is, B, weight_bytes):
    """Limit of the workgroups of the second half of a shared expert on its own stream."""
    return _library().second_half(T, d, E, I, Is, ctypes.c_longlong(B), weight_bytes)


def first_half_beside_route(T, d, E, I, Is, B, fp8):
    """Whether the shared expert's first half is part of the routing launch."""
    return bool(_library().beside_route(T, d, E, I, Is, ctypes.c_longlong(B), int(fp8)))


def dense_tile_rows(rows, col_tiles, most):
    return _library().tile_rows(ctypes.c_longlong(rows), col_tiles, ctypes.c_longlong(most))


def choice_of(w, budget=None):
    return choose(w.T, w.d, w.E, w.I, w.I_shared, w.budget if budget is None else budget)
