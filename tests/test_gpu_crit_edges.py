"""Critical values and histograms at the sizes where k_crit changes its path
(few keys, keys beyond the registers, few and many segments) and on values
that crowd or spread its intervals, against a sort."""
from __future__ import annotations

import math

import numpy as np
import pytest

from test_gpu_scan import fc, to_dev  # noqa: F401  (fc: fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ALPHA = (1e-9, 0.1, 0.5, 0.6827, 0.9, 0.95, 0.999, 1.0)


def values(kind, K, rng):
    if kind == "chi2":
        return rng.chisquare(2, K)
    if kind == "zeros":       # most values equal, the rest around them
        return np.where(rng.random(K) < 0.7, 0.0, rng.chisquare(2, K))
    if kind == "one_ulp":     # neighbouring doubles
        return np.nextafter(1.0, 2.0) * (1.0 + 2.0 ** -52 * rng.integers(0, 3, K))
    if kind == "wide":        # both signs, 600 orders of magnitude, NaN and infinities
        x = rng.choice([-1.0, 1.0], K) * 10.0 ** rng.uniform(-307, 307, K)
        x[rng.random(K) < 0.05] = np.nan
        x[rng.random(K) < 0.05] = np.inf
        x[rng.random(K) < 0.05] = -np.inf
        x[rng.random(K) < 0.05] = -0.0
        x[rng.random(K) < 0.05] = 5e-324
        return x
    return np.full(K, 3.25)   # "equal"


def key(x):
    """The order k_crit sorts by: numeric, -0 before +0, NaN last."""
    b = np.ascontiguousarray(x, dtype=np.float64).view(np.uint64)
    k = np.where(b >> np.uint64(63), ~b, b | np.uint64(1 << 63))
    return np.where(np.isnan(x), np.uint64(2 ** 64 - 1), k)


@pytest.mark.parametrize("kind", ["chi2", "zeros", "one_ulp", "wide", "equal"])
@pytest.mark.parametrize("sizes", [
    (0, 1, 2, 255, 256, 257), (1024, 1025, 20479, 20480, 20481), (50000,),
    tuple([3, 256, 257, 600] * 129), tuple([2559, 2560, 2561, 2700] * 129)])
def test_order_statistics_and_histogram(fc, kind, sizes):  # noqa: F811
    rng = np.random.default_rng([len(sizes), sizes[-1]])
    x = np.concatenate([values(kind, K, rng) for K in sizes])
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = len(sizes)
    crit = torch.full((n, len(ALPHA)), -7.0, dtype=torch.float64, device="cuda")
    hist = torch.full((n, 201), -7, dtype=torch.int64, device="cuda")
    fc.fc_critical_value(to_dev(off, torch.int64), to_dev(x, torch.float64), ALPHA, crit, 200, 50.0,
                         hist)
    torch.cuda.synchronize()
    crit, hist = crit.cpu().numpy(), hist.cpu().numpy()
    for s, K in enumerate(sizes):
        seg = x[off[s]:off[s + 1]]
        if K == 0:
            assert np.all(np.isnan(crit[s])) and not hist[s].any()
            continue
        order = seg[np.argsort(key(seg), kind="stable")]
        want = [order[min(max(math.ceil(a * K), 1), K) - 1] for a in ALPHA]
        assert np.array_equal(crit[s], want, equal_nan=True)
        inside = (seg >= 0.0) & (seg < 50.0)
        b = np.minimum(np.floor(seg[inside] / (50.0 / 200)), 199).astype(np.int64)
        h = np.bincount(b, minlength=201)
        h[200] += K - inside.sum()
        assert np.array_equal(hist[s], h)
