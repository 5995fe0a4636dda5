"""Searches over several bidders at once that end before all of them are placed (no GPU).

The rule of csrc/search_words.h for what is still to rise is tried on the CPU on searches that end after some of their paths; left out, rows
hold columns that are worth less to them than others by more than epsilon."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2303_13803_amd", "csrc")


@pytest.fixture(scope="module")
def searches(tmp_path_factory):
    program = str(tmp_path_factory.mktemp("search_end") / "search_end")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", CSRC, "-o", program, os.path.join(HERE, "search_end.cpp")], check=True)
    return lambda *a: subprocess.run([program, *a], capture_output=True, text=True, timeout=120)


def test_everybody_is_within_epsilon_of_the_best(searches):
    done = searches()
    assert done.returncode == 0, done.stdout


def test_not_if_the_other_trees_are_left_as_they_are(searches):
    done = searches("left out")
    assert done.returncode == 1, done.stdout
