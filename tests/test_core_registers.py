"""What the compiler keeps in memory for want of registers in the kernels of the phases on lists (no GPU).

Those kernels are bound by latency, and a value that does not fit a register is a trip to memory.  One wavefront more a SIMD is not worth
it where LDS does not let it in."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2303_13803_amd", "csrc")


@pytest.mark.skipif(not shutil.which("hipcc"), reason="no hipcc")
def test_registers_of_the_kernels_on_lists(tmp_path):
    done = subprocess.run(["hipcc", "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-w", "-I", CSRC,
                           "-I", os.path.join(CSRC, "..", "..", "include"), "--cuda-device-only", "-S", "-o", str(tmp_path / "core.s"), os.path.join(CSRC, "core.hip"),
                           "-Rpass-analysis=kernel-resource-usage"], capture_output=True, text=True, timeout=600, check=True)
    spilled = {}
    for name, rest in re.findall(r"Function Name: (\S+)(.*?)(?=Function Name:|\Z)", done.stderr, re.S):
        spilled[name] = int(re.search(r"VGPRs Spill: (\d+)", rest).group(1))
    engine = [n for k, n in spilled.items() if "core_kernel" in k]
    assert len(engine) == 2 and max(engine) <= 51, spilled
    lists = [n for k, n in spilled.items() if "core_list_kernel" in k]
    assert len(lists) == 3 and max(lists) == 0, spilled
