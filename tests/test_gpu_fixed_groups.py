"""One-matrix scans whose rounds mix the three launches (groups with a table,
tiles of at most 32 and of at most 16), each with its own grid chunks, on grids
of one, a few and many steps: every universe's results are those of its group
alone, bit for bit, and a sample equals the oracle's."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import parity
from test_gpu_fixed import run_fixed
from test_gpu_scan import FORM, fc  # noqa: F401  (fc: fixture)
from test_gpu_tile_edges import small_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,G", [(3, 20011), (5, 1), (21, 64), (38, 130), (57, 4099)])
@pytest.mark.parametrize("sizes", [(20,) + (1,) * 90, (300, 17, 1, 16), (5, 257, 32, 33, 64)])
def test_mixed_launches(fc, N, G, sizes):  # noqa: F811
    S, F, _, _ = small_problem(N, G, 1, 9)
    rng = np.random.default_rng([N, G, len(sizes)])
    sizes = sizes[:G]
    p = np.repeat(rng.choice(G, len(sizes), replace=False), sizes)
    p = p[rng.permutation(p.size)]
    d = S[p] + rng.standard_normal((p.size, N)) * np.sqrt(S[p])
    d[3 % p.size, 0] = np.nan                   # no chi2 below +inf
    g = fc.fc_build_grid([np.arange(G, dtype=float)], S)
    fc.fc_build_covariance(g, F, forms=FORM["fp64"])
    dev = run_fixed(fc, g, d, p, 2)
    for q in np.unique(p)[:6]:
        u = np.nonzero(p == q)[0]
        one = run_fixed(fc, g, d[u], p[u], 2)
        for k in dev:
            assert np.array_equal(dev[k][u], one[k], equal_nan=True), (k, q)
    u = rng.choice(p.size, min(p.size, 12), replace=False)
    u = u[~np.isnan(d[u, 0])]
    ref = oracle.scan_fixed_m(S, F, d[u], p[u], 2)
    scale = np.maximum(1.0, ref["chi2_p"])
    assert np.all(np.abs(dev["dchi2"][u] - ref["dchi2"]) <= parity.TOL["fp64"] * scale)
    for k in ("argmin", "m_final", "iters"):
        assert np.array_equal(dev[k][u], ref[k]), k
