"""Which entries of a line are looked at exactly when its list is made (no GPU).

csrc/list_cut.h is compiled for the CPU: of entries on, above and below cuts of either sign, with weights, K and duals up
to the largest there are, none worth its cut may be left out, and none far below it let through."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2303_13803_amd", "csrc")


def test_floats_leave_out_nothing_that_is_worth_the_cut(tmp_path):
    program = str(tmp_path / "list_cut")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", CSRC, "-o", program, os.path.join(HERE, "list_cut.cpp")], check=True)
    done = subprocess.run([program], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0 and ", 0 wrong" in done.stdout, done.stdout
