"""Draws by a row's runs (csrc/run_draw.h), the same code compiled for the host: a helper of the greedy builder, the row in LDS, draws what a
wave of the tree's workgroup draws from memory, bit for bit, and starts from the same totals."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("run_draw") / "check")
    clang = shutil.which("amdclang++") or "/opt/rocm/llvm/bin/clang++"          # (address spaces, vector types)
    subprocess.check_call([clang, "-std=c++17", "-O1", "-U_FORTIFY_SOURCE", "-Wall", "-Werror", "-I", os.path.join(HERE, "wave_on_host"), "-o", exe,
                           os.path.join(HERE, "run_draw_check.cpp")])
    return exe


@pytest.mark.parametrize("what,trials,seed", [("totals", 50, 1), ("draws", 130, 1), ("draws", 130, 5001)])
def test_a_helper_draws_what_the_nodes_own_wave_draws(check, what, trials, seed):
    r = subprocess.run([check, what, str(trials), str(seed)], capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, r.stdout
