"""The counter behind the partial records tells which workgroup of a launch merges them.  Calls that overlap on one
workspace race, but only they may be wrong: every order of two such launches on one counter word is walked on the CPU, and
from every value they can leave, every order of the launch that follows (the rules are the kernel's own header)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2502_15075_amd", "csrc")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("merge") / "merge_count_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, "-o", exe, os.path.join(HERE, "merge_count_check.cpp")], check=True)
    return lambda *a: subprocess.run([exe, *a], capture_output=True, text=True)


def test_a_launch_counts_right_whatever_overlapping_launches_left(check):
    r = check()
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[0].split("=")[1]) > 40


def test_the_walk_finds_the_fault_of_one_mark_for_all_launches(check):
    r = check("one")
    assert r.returncode == 1 and "wrong=0" not in r.stdout, r.stdout
