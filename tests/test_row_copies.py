"""The greedy builder's drawing waves keep copies of row totals (csrc/row_copies.h).  The same code, compiled for
the host: over random orders of service every draw must start from its row as the earlier draws left it."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("row_copies") / "check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-o", exe, os.path.join(HERE, "row_copies_check.cpp")])
    return exe


# trees smaller than the number of waves, with one and two nodes for some wave, and long after that
@pytest.mark.parametrize("rows", [1, 2, 13, 14, 15, 16, 28, 29, 32, 43, 64, 200])
@pytest.mark.parametrize("waves", [1, 3, 14])
def test_every_draw_knows_the_earlier_draws(check, rows, waves):
    r = subprocess.run([check, str(rows), str(waves), "400", str(1000 * rows + waves)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
