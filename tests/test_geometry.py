"""CPU checks of the launch geometry (compiled host-only from the library's own
headers): the scans' chunk counts against a search of all of them, their
limits, and the universe tiles of the fullest XCD against the kernel's own
assignment; the one-matrix scan's batches, tiles and candidate scratch."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.parametrize("name", ["geometry_check", "fixed_plan_check"])
def test_launch_plans(tmp_path, name):
    exe = tmp_path / name
    cmd = ["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
           "-I", os.path.join(ROOT, "paper_2002_07858_amd", "csrc"),
           os.path.join(HERE, name + ".cpp"), "-o", str(exe)]
    try:
        subprocess.check_call(cmd)
    except FileNotFoundError:
        pytest.skip("g++ not available")
    out = subprocess.run([str(exe)], capture_output=True, text=True).stdout
    assert out.strip().endswith("ok"), out
