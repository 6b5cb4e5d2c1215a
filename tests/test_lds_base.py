"""The tile kernel's loads into LDS take their destination from M0, written by a statement of its own
a few instructions earlier: whatever else writes M0 in between, the load gets its own base."""
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_08133_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SOURCE = """
#include <hip/hip_runtime.h>
#include "ffn_bf16_t256_kernel.hpp"
using namespace allocmoe;
__global__ void probe(const bf16x8* g, uint32_t first, uint32_t second) {
    const LdsBase a = set_lds_base(__builtin_amdgcn_readfirstlane(first));
    MIDDLE
    load_rows_to_lds(g + threadIdx.x, a);
}
"""
MIDDLES = {
    "nothing": "",
    "a clobber": 'asm volatile("s_mov_b32 m0, 0x1234" : : : "m0");',
    "another base": "const LdsBase b = set_lds_base(__builtin_amdgcn_readfirstlane(second)); load_rows_to_lds(g, b);",
}


@pytest.mark.parametrize("middle", MIDDLES)
def test_load_uses_its_own_base(tmp_path, middle):
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(SOURCE.replace("MIDDLE", MIDDLES[middle]))
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "--cuda-device-only", "-S", "-I", CSRC,
                           str(src), "-o", str(out)], stderr=subprocess.DEVNULL)
    code = [line.strip() for line in out.read_text().splitlines() if re.match(r"\t[a-z]", line)]
    # follow M0 (and copies of it) from write to write: the last load must see the first base
    holds, value = {"m0": None}, None
    writes = 0
    for line in code:
        m = re.match(r"s_mov_b32 (\w+), (\w+)", line)
        if m:
            to, src_reg = m.groups()
            if to == "m0" and src_reg not in holds:
                writes += 1
                holds["m0"] = writes if src_reg.startswith("s") else "other"
            else:
                holds[to] = holds.get(src_reg)
        if line.startswith("global_load_lds"):
            value = holds["m0"]
    assert value == 1, code
