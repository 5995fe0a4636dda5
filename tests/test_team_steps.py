"""Workgroups that work together come to the same decisions, also one that is held up after a barrier (no GPU).

csrc/team_steps.h is compiled for the CPU and run on threads.  The rules it replaces have to come apart
under the same schedules, or these would not be those that matter."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2303_13803_amd", "csrc")


@pytest.fixture(scope="module")
def steps(tmp_path_factory):
    program = str(tmp_path_factory.mktemp("team_steps") / "team_steps")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-pthread", "-I", CSRC, "-o", program,
                    os.path.join(HERE, "team_steps.cpp")], check=True)
    return lambda rule: subprocess.run([program, rule], capture_output=True, text=True, timeout=120)


def test_served_trees_get_their_labels_the_same_way_everywhere(steps):
    done = steps("labels")
    assert done.returncode == 0, done.stdout


def test_a_count_read_behind_the_barrier_sends_members_to_different_barriers(steps):
    done = steps("labels read late")
    assert done.returncode == 1 and int(done.stdout.split(" together, ")[1].split()[0]) > 0, done.stdout


def test_stages_go_on_from_the_same_counts_everywhere(steps):
    done = steps("stages")
    assert done.returncode == 0, done.stdout


@pytest.mark.parametrize("rule", ["stages begin anew", "cleared when read"])
def test_counts_cleared_before_everybody_has_read_them(steps, rule):
    done = steps(rule)
    assert done.returncode == 1 and int(done.stdout.split(" together, ")[1].split()[0]) > 0, done.stdout
