"""The scans at the edges of their tilings: bin counts at the borders of the
kernels' row groups and of the factorisation's tiles, universe counts at the
borders of their tiles, grids of one, two and a few points, against the FP64 oracle (tolerances of the forms,
as everywhere)."""
from __future__ import annotations

import time

import numpy as np
import pytest

import oracle
import parity
from test_gpu_fixed import run_fixed
from test_gpu_scan import FORM, fc, run_scan, to_dev  # noqa: F401  (fc: fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def small_problem(N, G, K, seed):
    """A smooth one-axis grid of G points and K universes at random true points."""
    rng = np.random.default_rng([seed, N, G, K])
    base = rng.uniform(80.0, 300.0, N)
    S = base + np.linspace(0.0, 1.0, G)[:, None] * rng.uniform(0.0, 30.0, N)
    A = rng.standard_normal((N, 2 * N))
    F = 0.01 * (A @ A.T) / (2 * N)
    F = 0.5 * (F + F.T)
    p = np.sort(rng.integers(0, G, K))
    d = S[p] + rng.standard_normal((K, N)) * np.sqrt(S[p])
    return S, F, p, d


def check(out, ref, S, F, d, p, tol):
    assert np.all(np.abs(out["dchi2"] - ref["dchi2"]) <= tol * np.maximum(1.0, ref["chi2_p"]))
    assert np.all(np.abs(out["chi2_p"] - ref["chi2_p"]) <= tol * np.maximum(1.0, ref["chi2_p"]))
    clear = ref["chi2_2nd"] - ref["chi2_min"] > 2 * tol * np.maximum(1.0, ref["chi2_min"])
    assert np.array_equal(out["argmin"][clear], ref["argmin"][clear])


# bin blocks of four in row groups of four blocks, with no, one and two lead bins
@pytest.mark.parametrize("N", [1, 2, 4, 5, 6, 16, 17, 18, 20, 21, 33, 36, 37, 49, 53, 58, 64])
@pytest.mark.parametrize("K,G", [(1, 1), (31, 2), (33, 3), (127, 7), (129, 5)])
def test_fp64_tiles_and_groups(fc, N, K, G):  # noqa: F811
    S, F, p, d = small_problem(N, G, K, 1)
    g = fc.fc_build_grid([np.arange(G, dtype=float)], S)
    fc.fc_build_covariance(g, F, forms=FORM["fp64"])
    ref = oracle.scan(S, F, d, p)
    check(run_scan(fc, g, FORM["fp64"], d, p), ref, S, F, d, p, parity.TOL["fp64"])


# groups of one matrix at the borders of the tiles (16, 32) and of the rule
# between on-the-fly and tabulated points (256), several groups a call
@pytest.mark.parametrize("N", [1, 4, 5, 16, 17, 32, 33, 48, 57, 64])
@pytest.mark.parametrize("iters", [0, 5])
def test_fixed_matrix_groups(fc, N, iters):  # noqa: F811
    sizes = (1, 16, 17, 33, 256, 257, 2)
    G = 77  # not a multiple of 16 or 64
    S, F, _, _ = small_problem(N, G, 1, 3)
    rng = np.random.default_rng([N, iters])
    p = np.repeat(np.sort(rng.choice(G, len(sizes), replace=False)), sizes)
    p = p[rng.permutation(p.size)]
    d = S[p] + rng.standard_normal((p.size, N)) * np.sqrt(S[p])
    g = fc.fc_build_grid([np.arange(G, dtype=float)], S)
    fc.fc_build_covariance(g, F, forms=FORM["fp64"])
    dev = run_fixed(fc, g, d, p, iters)
    ref = oracle.scan_fixed_m(S, F, d, p, iters)
    scale = np.maximum(1.0, ref["chi2_p"])
    assert np.all(np.abs(dev["dchi2"] - ref["dchi2"]) <= parity.TOL["fp64"] * scale)
    for k in ("argmin", "m_final", "iters"):
        assert np.array_equal(dev[k], ref[k]), k


# universes drawn in tiles that straddle segments and calls: one call of many
# short segments against the oracle's counts and against calls of one segment
@pytest.mark.parametrize("N", [1, 7, 57, 64])
def test_universe_tiles(fc, N):  # noqa: F811
    sizes = (1, 2, 15, 16, 17, 0, 5, 33, 4, 3000)
    S, F, _, _ = small_problem(N, len(sizes), 1, 4)
    S[3] *= 0.02  # means below 10: the other Poisson method
    g = fc.fc_build_grid([np.arange(len(sizes), dtype=float)], S)
    fc.fc_build_covariance(g, F, forms=FORM["fp32"])

    def draw(pts, lens):
        K = int(np.sum(lens))
        d = torch.empty((K, N), dtype=torch.float64, device="cuda")
        c = torch.empty((K, N), dtype=torch.int32, device="cuda")
        p = torch.empty(K, dtype=torch.int64, device="cuda")
        off = to_dev(np.concatenate([[0], np.cumsum(lens)]), torch.int64)
        fc.fc_generate_universes(g, to_dev(pts, torch.int64), off, 11, d, p, c)
        torch.cuda.synchronize()
        return d.cpu().numpy(), p.cpu().numpy(), c.cpu().numpy()

    pts = np.arange(len(sizes))
    d, p, c = draw(pts, sizes)
    assert np.array_equal(p, np.repeat(pts, sizes))
    lo = 0
    for q, n in zip(pts, sizes):
        if n == 0:
            continue
        one, _, one_c = draw(np.array([q]), (n,))
        assert np.array_equal(d[lo:lo + n], one) and np.array_equal(c[lo:lo + n], one_c)
        ref, ref_c = oracle.universes(S, F, [int(q)], [0, n], 11)
        assert np.array_equal(c[lo:lo + n], ref_c)
        # a sum of at most 64 terms below 1e3, log and cos within an ulp or two
        assert np.allclose(d[lo:lo + n], ref, rtol=0, atol=64 * 1e3 * 2.0 ** -50)
        lo += n


# covariances at the borders of the factorisation's tiles (16 rows) and panels
# (4 columns): W^T W against LAPACK's inverse, and a zero pivot in the
# first and the last bin found at its point
@pytest.mark.parametrize("N", [1, 2, 4, 15, 16, 17, 31, 32, 33, 44, 47, 48, 49, 57, 60, 63, 64])
def test_covariance_tiles(fc, N):  # noqa: F811
    G = 9
    S, F, _, _ = small_problem(N, G, 1, 5)
    stat = np.linspace(20.0, 500.0, N)
    g = fc.fc_build_grid([np.arange(G, dtype=float)], S)
    fc.fc_build_covariance(g, F, fc.FC_STAT_FIXED, stat, forms=FORM["fp64"])
    out = torch.empty((G, N, N), dtype=torch.float64, device="cuda")
    fc.fc_grid_inverse_cov(g, 0, G, out)
    torch.cuda.synchronize()
    for q in range(G):
        sig = oracle.covariance(S[q], F, oracle.STAT_FIXED, stat)
        ref = np.linalg.inv(sig)
        err = np.linalg.norm(out[q].cpu().numpy() - ref) / np.linalg.norm(ref)
        assert err <= 1e-12 * np.linalg.cond(sig), (q, err)
    for b in {0, N - 1}:
        Z = S.copy()
        Z[4:, b] = 0.0
        g = fc.fc_build_grid([np.arange(G, dtype=float)], Z)
        with pytest.raises(fc.FCError) as ei:
            fc.fc_build_covariance(g, F, fc.FC_STAT_FIXED, np.zeros(N), forms=FORM["fp64"])
        assert ei.value.code == fc.FC_ERR_NOT_PD and ei.value.bad_q == 4


# served requests whose items are cut to the least length, to one in between
# and to the largest, on grids of less than one item, of one, and with a
# remainder: bit for bit fc_scan's results
@pytest.mark.parametrize("form", ["fp32", "split_bf16", "split_fp16"])
@pytest.mark.parametrize("G,sizes", [(1, (1, 300)), (31, (1,)), (33, (255, 257)), (129, (1, 2, 3)),
                                     (5000, (1, 700)), (20011, (5000, 1, 3000)), (70001, (31000, 1))])
def test_served_items(fc, form, G, sizes):  # noqa: F811
    N = 19
    S, F, p, d = small_problem(N, G, sum(sizes), 6)
    g = fc.fc_build_grid([np.arange(G, dtype=float)], S)
    fc.fc_build_covariance(g, F, forms=FORM[form])
    srv = fc.Server([g], form=FORM[form], hbm_budget=64 << 20, host_budget=64 << 20)
    try:
        lo, ids = 0, []
        for n in sizes:
            ids.append(srv.submit(0, int(p[lo]), d[lo:lo + n]))
            lo += n
        lo = 0
        for i, n in zip(ids, sizes):
            state, got = srv.poll(i)
            while got is None:
                assert state != fc.FC_REQ_FAILED
                time.sleep(1e-4)
                state, got = srv.poll(i)
            ref = run_scan(fc, g, FORM[form], d[lo:lo + n], np.full(n, p[lo]))
            for k in ("dchi2", "chi2_min", "argmin", "chi2_p"):
                assert np.array_equal(got[k], ref[k]), (n, k)
            lo += n
    finally:
        srv.destroy()
