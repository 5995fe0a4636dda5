"""The two best values of half a list, found by float distances and settled in doubles (no GPU).

csrc/half_list.h is compiled for the CPU and run with arrays in a wavefront's place, from small whole numbers with many
ties to numbers of 2^50 that differ by one.  The second value taken from its float, rounded up, has to
fail where floats no longer tell whole numbers apart."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2303_13803_amd", "csrc")


@pytest.fixture(scope="module")
def half(tmp_path_factory):
    program = str(tmp_path_factory.mktemp("half_list") / "half_list")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", CSRC, "-o", program, os.path.join(HERE, "half_list.cpp")], check=True)
    return lambda rule: subprocess.run([program, rule], capture_output=True, text=True, timeout=120)


def test_the_two_best_are_exact(half):
    done = half("exact")
    assert done.returncode == 0, done.stdout


def test_a_second_value_from_its_float_is_not(half):
    done = half("rounded up")
    assert done.returncode == 1 and ", 0 wrong lanes" in done.stdout, done.stdout
