"""Draws without replacement by one wave (csrc/wave_draw.h), the same code compiled for the host: it stays inside the row's LDS also
where the weights are infinite, and the quick step with its retry draws what the exact form draws, bit for bit."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("wave_draw") / "check")
    clang = shutil.which("amdclang++") or "/opt/rocm/llvm/bin/clang++"          # (address spaces, vector types)
    subprocess.check_call([clang, "-std=c++17", "-O1", "-U_FORTIFY_SOURCE", "-Wall", "-Werror", "-I", os.path.join(HERE, "wave_on_host"), "-o", exe,
                           os.path.join(HERE, "wave_draw_check.cpp")])
    return exe


# rows that end in a leaf, a group, the last group, and just past each
@pytest.mark.parametrize("V", [1, 31, 32, 33, 511, 512, 513, 1000, 16384, 16385, 32000, 32255, 32256, 32257, 32737, 32768])
def test_draws_of_infinite_weight_stay_in_the_row(check, V):
    r = subprocess.run([check, "range", str(V)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("seed", [1, 10001])
def test_quick_step_and_retry_draw_what_the_exact_form_draws(check, seed):
    r = subprocess.run([check, "exact", "200", str(seed)], capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, r.stdout
