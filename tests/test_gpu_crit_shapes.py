"""Critical values and histograms in each block shape of k_crit (up to 256
segments, up to 512, more), with few bins and near the limit of 16 383, whose
counters take 64 KiB of LDS beside the kernel's own, against a sort."""
from __future__ import annotations

import math

import numpy as np
import pytest

from test_gpu_crit_edges import ALPHA, key, values
from test_gpu_scan import fc, to_dev  # noqa: F401  (fc: fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n_bins", [1, 16383])
@pytest.mark.parametrize("kind", ["zeros", "wide"])
@pytest.mark.parametrize("n_seg", [3, 256, 257, 512, 513])
def test_block_shapes(fc, n_seg, kind, n_bins):  # noqa: F811
    rng = np.random.default_rng([n_seg, n_bins])
    sizes = rng.choice([0, 1, 63, 255, 256, 257, 300, 1100], n_seg)
    sizes[1] = 10241      # more than the registers of 512 threads hold
    x = np.concatenate([values(kind, K, rng) for K in sizes])
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    crit = torch.full((n_seg, len(ALPHA)), -7.0, dtype=torch.float64, device="cuda")
    hist = torch.full((n_seg, n_bins + 1), -7, dtype=torch.int64, device="cuda")
    fc.fc_critical_value(to_dev(off, torch.int64), to_dev(x, torch.float64), ALPHA, crit, n_bins,
                         50.0, hist)
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
        b = np.minimum(np.floor(seg[inside] / (50.0 / n_bins)), n_bins - 1).astype(np.int64)
        h = np.bincount(b, minlength=n_bins + 1)
        h[n_bins] += K - inside.sum()
        assert np.array_equal(hist[s], h)
