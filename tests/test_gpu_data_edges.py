"""The data scan at the ends of its ranges: bin counts up to 64, grids from one
point to more than its blocks take at once, against a plain evaluation; and its
scratch, which must not come from the stream-ordered pool (the call waits, so
that the pool would be emptied and filled again by every call)."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

import oracle
import parity
from test_gpu_scan import FORM, fc, to_dev  # noqa: F401  (fc: fixture)
from test_gpu_tile_edges import small_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def hip():
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64.so" in line)
    return ctypes.CDLL(path)


def pool_peak(call):
    """Bytes of the device's default pool in use at most during call()."""
    lib, pool, high = hip(), ctypes.c_void_p(), ctypes.c_uint64(0)
    used_high = 8  # hipMemPoolAttrUsedMemHigh
    assert lib.hipDeviceGetDefaultMemPool(ctypes.byref(pool), 0) == 0
    assert lib.hipMemPoolSetAttribute(pool, used_high, ctypes.byref(high)) == 0
    call()
    torch.cuda.synchronize()
    assert lib.hipMemPoolGetAttribute(pool, used_high, ctypes.byref(high)) == 0
    return high.value


def test_data_scan_leaves_the_pool_alone(fc):  # noqa: F811
    S, F, p, d = small_problem(5, 9, 300, 1)
    g = fc.fc_build_grid([np.arange(9.0)], S, d[0])
    fc.fc_build_covariance(g, F, forms=FORM["fp64"] | FORM["fp32"])
    out = torch.empty(9, dtype=torch.float64, device="cuda")
    dd, pp = to_dev(d, torch.float64), to_dev(p, torch.int64)
    dchi2 = torch.empty(300, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    # a scan without outputs of its own does take pool memory
    assert pool_peak(lambda: fc.fc_scan(g, FORM["fp32"], dd, pp, dchi2)) > 0
    assert pool_peak(lambda: fc.fc_data_scan(g, out)) == 0


# the largest bin count's triangles take more than 64 KiB of LDS a block; grids
# of one point, of a block's points and around them, and of several rounds of
# resident blocks
@pytest.mark.parametrize("N", [1, 2, 33, 57, 63, 64])
@pytest.mark.parametrize("G", [1, 3, 4, 5, 9001])
def test_data_scan_sizes(fc, N, G):  # noqa: F811
    S, F, _, d = small_problem(N, G, 1, 2)
    g = fc.fc_build_grid([np.arange(G, dtype=float)], S, d[0])
    fc.fc_build_covariance(g, F, forms=FORM["fp64"])
    out = torch.full((G,), -7.0, dtype=torch.float64, device="cuda")
    low, at = fc.fc_data_scan(g, out)
    ref, rlow, rat = oracle.data_scan(S, F, d[0])
    scale = np.maximum(1.0, ref + rlow)
    assert np.all(np.abs(out.cpu().numpy() - ref) <= parity.TOL["fp64"] * scale)
    assert abs(low - rlow) <= parity.TOL["fp64"] * max(1.0, rlow)
    assert ref[at] <= 2 * parity.TOL["fp64"] * max(1.0, rlow)
