"""The rules by which the greedy builder uses its helpers' rings (csrc/helper_rings.h), the same code compiled for the host."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("helper_rings") / "check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-o", exe, os.path.join(HERE, "helper_rings_check.cpp")])
    return exe


def test_a_helper_that_runs_is_used_whatever_the_others_do(check):
    r = subprocess.run([check, "free"], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("seed", [1, 100001])
def test_a_nodes_draws_come_in_order_and_without_long_waits(check, seed):
    r = subprocess.run([check, "draws", "300", str(seed)], capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, r.stdout
