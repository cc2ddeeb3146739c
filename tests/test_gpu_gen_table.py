"""Universes of long segments, whose tiles take the squeeze's constants from a
table of the tile's first point, with short segments among them (tiles of several
points, first points outside the grid, means below 10), and universe counts on
both sides of where a tile gets another row: counts equal to the oracle's, rows
of a point equal to a call of that point alone."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from test_gpu_gen_tiles import draw
from test_gpu_scan import FORM, fc  # noqa: F401  (fc: fixture)
from test_gpu_tile_edges import small_problem

pytestmark = pytest.mark.gpu

G = 12


def check(fc, N, pts, lengths):  # noqa: F811
    S, F, _, _ = small_problem(N, G, 1, 17)
    S[::5] *= 0.02
    g = fc.fc_build_grid([np.arange(G, dtype=float)], S)
    fc.fc_build_covariance(g, F, forms=FORM["fp32"])
    off = np.concatenate([[0], np.cumsum(lengths)])
    d, p, c = draw(fc, g, N, np.array(pts), off, 29)
    for s, pt in enumerate(pts):
        lo, hi = int(off[s]), int(off[s + 1])
        if lo == hi:
            continue
        if not 0 <= pt < G:
            assert np.all(p[lo:hi] == -1)
            assert np.all(np.isnan(d[lo:hi])) and np.all(c[lo:hi] == -1)
            continue
        assert np.all(p[lo:hi] == pt)
        one, _, one_c = draw(fc, g, N, np.array([pt]), np.array([0, hi - lo]), 29)
        assert np.array_equal(d[lo:hi], one) and np.array_equal(c[lo:hi], one_c)
        n = min(hi - lo, 40)
        _, ref = oracle.universes(S, F, [pt], [0, n], 29)
        assert np.array_equal(c[lo:lo + n], ref)


@pytest.mark.parametrize("N", [17, 57, 64])
@pytest.mark.parametrize("scale", [1, 8])
def test_short_segments_among_long(fc, N, scale):  # noqa: F811
    check(fc, N, [3, 5, -1, 5, 7, 0, G, 4, 3], [1501 * scale, 1, 3, 2, 5, 2002 * scale, 3, 0, 900])


@pytest.mark.parametrize("K", [447, 448, 703, 704, 959, 960, 3072, 3073])
def test_rows_a_tile(fc, K):  # noqa: F811
    check(fc, 57, [5, 2], [K - 9, 9])
