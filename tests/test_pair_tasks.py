"""Tasks of the pair kernel are dealt out once each, and there are enough of them (no GPU): csrc/pair_tasks.h compiled for the CPU."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2303_13803_amd", "csrc")


def test_tasks_of_the_pair_kernel(tmp_path):
    program = str(tmp_path / "pair_tasks")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", CSRC, "-o", program, os.path.join(HERE, "pair_tasks.cpp")], check=True)
    done = subprocess.run([program, "2000", "1"], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, done.stdout
