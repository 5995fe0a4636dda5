"""What wavefronts that scan one row in the same step leave behind, in every order (no GPU).

csrc/search_words.h holds what a search on lists publishes of a scan and what the pass over all
columns concludes from it; tests/search_words.cpp compiles those functions for the CPU and tries all
orders of their memory accesses.  The same orders with plain stores in the place of the minima have
to show the fault, or the check would be worth nothing."""
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2303_13803_amd", "csrc")


@pytest.fixture(scope="module")
def orders(tmp_path_factory):
    program = str(tmp_path_factory.mktemp("search_words") / "search_words")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", CSRC, "-o", program, os.path.join(HERE, "search_words.cpp")],
                   check=True)

    def run(*args):
        out = subprocess.run([program, *args], check=True, capture_output=True, text=True).stdout
        return {what: (int(n), int(bad)) for what, n, bad in re.findall(r"(.+): (\d+) orders, (\d+) broken", out)}
    return run


def test_scans_of_one_row_in_any_order(orders):
    tried, broken = orders()["scans"]
    assert tried > 1000 and broken == 0
    assert orders("stores")["scans"][1] > 0


def test_a_line_read_whole_while_its_row_is_scanned(orders):
    """Nothing unlisted is hidden, whichever labels the slices of the line and the scans read, and a line whose
    label has not moved is not asked for a second time."""
    tried, broken = orders()["whole lines"]
    assert tried > 1000 and broken == 0
    assert orders("stores")["whole lines"][1] > 0 and orders("moved")["whole lines"][1] > 0
