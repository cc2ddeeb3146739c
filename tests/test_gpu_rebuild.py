"""A grid rebuilt with other matrices and other forms gives what a fresh grid
gives, and a rebuild waits for scans still running on another stream."""
from __future__ import annotations

import numpy as np
import pytest

import fcgen
from test_gpu_scan import FORM, fc, run_scan, to_dev  # noqa: F401  (fc: fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sequence", [("fp64", "fp64"), ("fp32", "split_fp16", "fp32"),
                                      ("fp64", "fp32", "fp64"), ("split_bf16", "fp64")])
def test_rebuild_equals_fresh_grid(fc, sequence):  # noqa: F811
    pr = fcgen.make_problem("c1", K=200)
    g = fc.fc_build_grid(pr.axes, pr.S)
    for k, form in enumerate(sequence):
        F = pr.F * (1.0 + 0.5 * k)
        stat = None if k % 2 == 0 else np.linspace(50.0, 90.0, pr.N)
        mode = fc.FC_STAT_PEARSON if stat is None else fc.FC_STAT_FIXED
        fc.fc_build_covariance(g, F, mode, stat, forms=FORM[form])
        fresh = fc.fc_build_grid(pr.axes, pr.S)
        fc.fc_build_covariance(fresh, F, mode, stat, forms=FORM[form])
        assert fc.fc_grid_device_bytes(g) == fc.fc_grid_device_bytes(fresh)
        assert fc.fc_grid_info(g)["forms"] == FORM[form]
        a, b = (run_scan(fc, x, FORM[form], pr.d, pr.p_idx) for x in (g, fresh))
        assert all(np.array_equal(a[n], b[n]) for n in a)


def test_failed_rebuild_keeps_no_form_and_the_grid_builds_again(fc):  # noqa: F811
    pr = fcgen.make_problem("c1", K=50)
    g = fc.fc_build_grid(pr.axes, pr.S)
    fc.fc_build_covariance(g, pr.F, forms=FORM["fp64"])
    want = run_scan(fc, g, FORM["fp64"], pr.d, pr.p_idx)
    with pytest.raises(fc.FCError) as e:
        fc.fc_build_covariance(g, -np.eye(pr.N), forms=FORM["fp64"])
    assert e.value.code == fc.FC_ERR_NOT_PD and fc.fc_grid_info(g)["forms"] == 0
    fc.fc_build_covariance(g, pr.F, forms=FORM["fp64"])
    got = run_scan(fc, g, FORM["fp64"], pr.d, pr.p_idx)
    assert all(np.array_equal(want[n], got[n]) for n in want)


def test_rebuild_waits_for_a_scan_on_another_stream(fc):  # noqa: F811
    pr = fcgen.make_problem("c2", n_true=4, K=500)
    g = fc.fc_build_grid(pr.axes, pr.S)
    fc.fc_build_covariance(g, pr.F, forms=FORM["fp32"])
    want = run_scan(fc, g, FORM["fp32"], pr.d, pr.p_idx)
    d, p = to_dev(pr.d, torch.float64), to_dev(pr.p_idx, torch.int64)
    out = torch.empty(pr.K, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    for _ in range(4):
        fc.fc_scan(g, FORM["fp32"], d, p, out, stream=side)
    fc.fc_build_covariance(g, 2.0 * pr.F, forms=FORM["fp32"])  # on the current stream
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), want["dchi2"])
