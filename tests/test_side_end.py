"""When the sides of a phase that only prepares prices end, and what the next phases then have to do (no GPU).

csrc/side_end.h is compiled for the CPU and steers ladders of phases over weights that differ by a few units on top of a
large one, where every column too many has to come all the way down.  A limit on the steps of every side at every size leaves them all to
the first phase that runs to the end."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2303_13803_amd", "csrc")


@pytest.fixture(scope="module")
def ladder(tmp_path_factory):
    program = str(tmp_path_factory.mktemp("side_end") / "side_end")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-I", CSRC, "-o", program, os.path.join(HERE, "side_end.cpp")], check=True)
    return lambda *a: subprocess.run([program, *map(str, a)], capture_output=True, text=True, timeout=120)


@pytest.mark.parametrize("n,m,base,spread", [(300, 330, 2 ** 29, 3), (900, 950, 2 ** 29, 3), (300, 600, 2 ** 29, 3), (300, 330, 2 ** 30, 0), (900, 965, 2 ** 29, 3), (300, 317, 2 ** 29, 3)])
def test_what_a_phase_leaves_to_the_next_is_bounded(ladder, n, m, base, spread):
    done = ladder(n, m, base, spread, "as it is")
    assert done.returncode == 0, done.stdout


@pytest.mark.parametrize("n,m", [(300, 330), (900, 950)])
def test_a_limit_on_the_steps_of_every_side_is_not(ladder, n, m):
    done = ladder(n, m, 2 ** 29, 3, "every side")
    assert done.returncode == 1, done.stdout


@pytest.mark.parametrize("phases,unasked", [(1, 3), (5, 3), (6, 4), (36, 4)])
def test_as_many_phases_run_to_the_end_as_are_asked_for(ladder, phases, unasked):
    """Also where that is as many as on longer ladders without being asked."""
    assert [int(ladder("asked", asked, phases).stdout) for asked in (0, 1, 3, 4, 5, 64)] == [unasked, 1, 3, 4, 5, 64]
