"""CPU check of the scans' launch geometry (compiled host-only from the
library's own header): the chunk counts chosen against a search of all of them,
their limits, and the universe tiles of the fullest XCD against the kernel's
own assignment."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_scan_geometry(tmp_path):
    exe = tmp_path / "geometry_check"
    cmd = ["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
           "-I", os.path.join(ROOT, "paper_2002_07858_amd", "csrc"),
           os.path.join(HERE, "geometry_check.cpp"), "-o", str(exe)]
    try:
        subprocess.check_call(cmd)
    except FileNotFoundError:
        pytest.skip("g++ not available")
    out = subprocess.run([str(exe)], capture_output=True, text=True).stdout
    assert out.strip().endswith("ok"), out
