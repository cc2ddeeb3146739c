"""Universes in tiles of several points, among them points outside the grid and
means below 10, at universe counts that take one row a tile, a few rows with at
most a draw a thread, and full tiles: counts equal to the oracle's, rows of a
point equal to a call of that point alone."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from test_gpu_scan import FORM, fc, to_dev  # noqa: F401  (fc: fixture)
from test_gpu_tile_edges import small_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def draw(fc, g, N, pts, off, seed):  # noqa: F811
    K = int(off[-1])
    d = torch.full((K, N), -7.0, dtype=torch.float64, device="cuda")
    c = torch.full((K, N), -7, dtype=torch.int32, device="cuda")
    p = torch.full((K,), -7, dtype=torch.int64, device="cuda")
    fc.fc_generate_universes(g, to_dev(pts, torch.int64), to_dev(off, torch.int64), seed, d, p, c)
    torch.cuda.synchronize()
    return d.cpu().numpy(), p.cpu().numpy(), c.cpu().numpy()


@pytest.mark.parametrize("N", [1, 19, 64])
@pytest.mark.parametrize("n_pts,most", [(5, 3), (300, 2), (1500, 3), (900, 40)])
def test_tiles_of_several_points(fc, N, n_pts, most):  # noqa: F811
    G = 40
    S, F, _, _ = small_problem(N, G, 1, 11)
    S[::7] *= 0.02
    g = fc.fc_build_grid([np.arange(G, dtype=float)], S)
    fc.fc_build_covariance(g, F, forms=FORM["fp32"])
    rng = np.random.default_rng([N, n_pts, most])
    pts = rng.integers(-1, G + 1, n_pts)        # -1 and G lie outside
    pts[:3] = (3, G, 7)
    off = np.concatenate([[0], np.cumsum(rng.integers(0, most + 1, n_pts))])
    d, p, c = draw(fc, g, N, pts, off, 13)
    inside = (pts >= 0) & (pts < G)
    assert np.array_equal(p, np.repeat(np.where(inside, pts, -1), np.diff(off)))
    for s in np.concatenate([np.arange(3), rng.choice(n_pts, 2)]):
        lo, hi = off[s], off[s + 1]
        if lo == hi:
            continue
        if not inside[s]:
            assert np.all(np.isnan(d[lo:hi])) and np.all(c[lo:hi] == -1)
            continue
        one, _, one_c = draw(fc, g, N, pts[s:s + 1], np.array([0, hi - lo]), 13)
        assert np.array_equal(d[lo:hi], one) and np.array_equal(c[lo:hi], one_c)
        _, ref = oracle.universes(S, F, [int(pts[s])], [0, int(hi - lo)], 13)
        assert np.array_equal(c[lo:hi], ref)
