"""The rings that the greedy builder's helpers write to (csrc/row_workspace.h), the same code compiled for the host: apart from all that the
tree's own waves keep in the workspace, for every size of tree that has helpers."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_the_rings_lie_apart(tmp_path):
    exe = str(tmp_path / "check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fno-strict-aliasing", "-Wall", "-Werror", "-o", exe, os.path.join(HERE, "mail_ring_check.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
