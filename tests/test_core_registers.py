"""What the compiler keeps in memory for want of registers in the kernels of the phases on lists and in the pair kernel (no GPU).

The kernels on lists are bound by latency, and a value that does not fit a register is a trip to memory.  One wavefront more a SIMD is not worth
it where LDS does not let it in."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2303_13803_amd", "csrc")


def _spilled(source, tmp_path):
    """Vector registers that each kernel of a source keeps in memory, by the kernel's mangled name."""
    done = subprocess.run(["hipcc", "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-w", "-I", CSRC,
                           "-I", os.path.join(CSRC, "..", "..", "include"), "--cuda-device-only", "-S", "-o", str(tmp_path / "kernels.s"), os.path.join(CSRC, source),
                           "-Rpass-analysis=kernel-resource-usage"], capture_output=True, text=True, timeout=600, check=True)
    return {name: int(re.search(r"VGPRs Spill: (\d+)", rest).group(1))
            for name, rest in re.findall(r"Function Name: (\S+)(.*?)(?=Function Name:|\Z)", done.stderr, re.S)}


@pytest.mark.skipif(not shutil.which("hipcc"), reason="no hipcc")
def test_registers_of_the_kernels_on_lists(tmp_path):
    spilled = _spilled("core.hip", tmp_path)
    engine = [n for k, n in spilled.items() if "core_kernel" in k]
    assert len(engine) == 2 and max(engine) == 0, spilled
    lists = [n for k, n in spilled.items() if "core_list_kernel" in k]
    assert len(lists) == 3 and max(lists) == 0, spilled


@pytest.mark.skipif(not shutil.which("hipcc"), reason="no hipcc")
def test_registers_of_the_pair_kernel(tmp_path):
    """What a task needs, and the index maps' rows, are kept in memory beside 64 projections and 128 accumulators; it is read between
    tasks, and where rows are scored as they come twice a row.  Hidden units, SM share, slowdown unit, fp16 pieces, long passes."""
    spilled = {re.search(r"pair_mlp_kernelILi(\d+)ELb(\d)ELb(\d)ELb(\d)ELb(\d)E", k).groups(): n
               for k, n in _spilled("score.hip", tmp_path).items() if "pair_mlp_kernel" in k}
    assert len(spilled) == 32
    for kind, most in ((("128", "0", "0", "1"), 13), (("64", "0", "0", "1"), 6), (("128", "1", "1", "1"), 27)):
        assert max(spilled[kind + (long,)] for long in "01") <= most, spilled
    assert max(n for k, n in spilled.items() if k[4] == "0") <= 19, spilled
    assert max(n for k, n in spilled.items() if k[0] == "64") <= 10, spilled
