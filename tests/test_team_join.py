"""Workgroups of launches that work together find each other, also beside another launch (no GPU).

csrc/team_join.h is compiled for the CPU and run on threads that stand for compute units.  Two launches
that each hold half of them, or a die each, would wait for one another's workgroups for ever: they have
to go on with the members they have.  Without that rule the same schedules end in waits that run out."""
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2303_13803_amd", "csrc")


@pytest.fixture(scope="module")
def join(tmp_path_factory):
    program = str(tmp_path_factory.mktemp("team_join") / "team_join")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-pthread", "-I", CSRC, "-o", program,
                    os.path.join(HERE, "team_join.cpp")], check=True)
    return lambda *args: subprocess.run([program, *map(str, args)], capture_output=True, text=True, timeout=120)


def test_two_launches_at_once_both_get_a_team(join):
    done = join(20000, 2000000000)
    assert done.returncode == 0, done.stdout


def test_without_closing_the_team_their_waits_run_out(join):
    done = join(2000000000, 300000)
    assert done.returncode == 1, done.stdout
    for launches in ("halves", "a die each"):
        assert sum(int(n) for n in re.findall(launches + r": \d+ members, (\d+) gave up", done.stdout)) > 0, done.stdout
