"""Whole lines read by several wavefronts: nobody waits for long (no GPU).

csrc/line_parts.h is compiled for the CPU and tried on all numbers of lines.  The rule for feasible prefixes, which leaves out parts that may be
empty, has to fail on lines that are whole."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2303_13803_amd", "csrc")


@pytest.fixture(scope="module")
def parts(tmp_path_factory):
    program = str(tmp_path_factory.mktemp("line_parts") / "line_parts")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", CSRC, "-o", program, os.path.join(HERE, "line_parts.cpp")], check=True)
    return lambda *rule: subprocess.run([program, *rule], capture_output=True, text=True, timeout=120)


def test_wavefronts_share_whole_lines_evenly(parts):
    done = parts()
    assert done.returncode == 0, done.stdout


def test_the_rule_for_prefixes_does_not(parts):
    done = parts("prefixes")
    assert done.returncode == 1, done.stdout
