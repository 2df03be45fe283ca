"""The greedy builder's workspace row (csrc/row_workspace.h), the same code compiled for the host: the draws that one node can see
and the one put aside have places of their own, for every size of tree."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_draws_of_one_node_have_places_of_their_own(tmp_path):
    exe = str(tmp_path / "check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fno-strict-aliasing", "-Wall", "-Werror", "-o", exe, os.path.join(HERE, "row_workspace_check.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
