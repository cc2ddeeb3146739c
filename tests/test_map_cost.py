"""CPU check of the covariance build's gather maps and of the time to fill them
(compiled host-only from the library's own header)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_gather_maps(tmp_path):
    exe = tmp_path / "map_cost_check"
    cmd = ["/opt/rocm/bin/hipcc", "-std=c++17", "-O3", "--offload-arch=gfx950", "-x", "hip",
           "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2002_07858_amd", "csrc"),
           os.path.join(HERE, "map_cost_check.cpp"), "-o", str(exe)]
    if not os.path.exists(cmd[0]):
        pytest.skip("hipcc not available")
    subprocess.check_call(cmd)
    out = subprocess.run([str(exe)], capture_output=True, text=True).stdout
    assert out.strip().endswith("ok"), out
