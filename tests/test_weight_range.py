"""Weight loads past the end of a stream (the kernels keep a fixed number of steps in flight) have to
be stopped by the buffer descriptor's range check, which covers the lane's offset and the
instruction's own; the scalar offset is documented as left out of it.  So no weight load may have one."""
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_08133_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SOURCES = {
    "streaming kernel": '#include "ffn_bf16.hip"',
}


@pytest.mark.parametrize("kernel", SOURCES)
def test_no_scalar_offset(tmp_path, kernel):
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(SOURCES[kernel])
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "--cuda-device-only", "-S", "-I", CSRC,
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", str(src), "-o", str(out)],
                          stderr=subprocess.DEVNULL)
    loads = re.findall(r"buffer_load_dwordx4 (.*)", out.read_text())
    assert loads
    for load in loads:   # destination, lane offset, descriptor, scalar offset and modifiers
        offset, modifiers = re.fullmatch(r"[av]\[\d+:\d+\], v\d+, s\[\d+:\d+\], (\S+) (.*)", load.strip()).groups()
        assert offset == "0" and modifiers.startswith("offen"), load
