"""The basis form (one pass over R shared by every point of a call) against the
FP64 oracle at the edges of its tiles: rows around the fold's stages of 32 and
quads of 4, bins around the 16-bin tiles, the 64-bin slices and the 256-column
fold tiles, points around the blocks of 16; several blocks per wave; more
analyses than one grouped launch takes.

Tolerance: the oracle sums nodes and rows directly, the basis form in another
order, so a mu_j differs by at most (rows + nodes + 128) roundings of 2^-53
relative (rel below).  -2lnL moves by 2 sum_j |mu_j - n_j| rel plus its own
summation, and the gradient by rel times the sum over bins of (|a_j| + 2 n_j /
mu_j) |d mu_j|, the latter bounded by the spectrum's change over a unit step
each way, with a factor of 8 for the two cancelling coupling terms."""
import numpy as np
import pytest

import synth
from problems import gpu_context, inputs

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -53
N_E = 24


def check(p, th, nll, grad, mu, pick):
    o, n, b = p["oracle"], p["n"], p["b"]
    rel = (p["n_t"] + 3 * N_E + 2 + 128) * EPS
    for i in pick:
        m, v, g = o.mu(th[i]), *o.nll_grad(th[i])
        assert np.all(np.abs(mu[i] - m) <= rel * np.abs(m)), i
        tol = 2 * np.abs(m - n).sum() * rel + 2 * (m + n).sum() * 64 * EPS
        assert abs(nll[i] - v) <= tol, (i, nll[i] - v, tol)
        w = np.abs(2 * (1 - n / m)) + 2 * n / m
        for k in range(7):
            d = np.zeros_like(m)
            for s in (-1.0, 1.0):
                t = th[i].copy()
                t[k] += s
                d += np.abs(o.mu(t) - m)
            assert abs(grad[i, k] - g[k]) <= 8 * rel * (w * d).sum(), (i, k)


@pytest.mark.parametrize("n_t,n_reco,n_pts", [
    (1, 1, 1), (31, 16, 15), (32, 17, 16), (33, 15, 17), (67, 127, 2), (96, 129, 33),
    (64, 255, 5), (129, 257, 1), (1030, 513, 48), (161, 4, 65)])
def test_edges_against_the_oracle(n_t, n_reco, n_pts):
    p = inputs(n_t, n_reco, N_E, 100_000, 8300 + n_t, 8301 + n_reco)
    ctx = gpu_context(p)
    th = synth.theta_prior(n_pts, 8302, f_range=(0.8, 1.2))
    nll, grad = ctx.eval_nll_grad(th)
    mu = ctx.eval_mu(th)
    check(p, th, nll, grad, mu, sorted({0, n_pts // 2, n_pts - 1}))
    # every entry point's likelihood is the same sum
    assert np.array_equal(ctx.eval_nll(th), nll)
    v, g = ctx.eval_nll_templates(th, grad=True)
    assert np.array_equal(v, nll) and np.array_equal(g, grad)
    ctx.set_band_skipping(True)
    assert np.array_equal(ctx.eval_nll(th), nll)
    ctx.close()


@pytest.mark.parametrize("n_pts", [4097, 32768 + 3, 65536])
def test_many_points_per_wave(n_pts):
    """Two and four blocks of points per wave: bitwise the lists' results,
    whose slices of 64 bins are the same."""
    import torch
    p = inputs(64, 512, N_E, 100_000, 8311, 8312)
    ctx = gpu_context(p)
    th = synth.theta_prior(n_pts, 8313, f_range=(0.8, 1.2))
    tt = torch.tensor(th, device="cuda:0")
    nll = torch.empty(n_pts, dtype=torch.float64, device="cuda:0")
    grad = torch.empty(n_pts, 7, dtype=torch.float64, device="cuda:0")
    ctx.build_templates()
    ctx.eval_nll_templates_dev(tt, nll, grad)
    torch.cuda.synchronize()
    nll, grad = nll.cpu().numpy(), grad.cpu().numpy()
    for a, b in ((0, 70), (n_pts // 2, n_pts // 2 + 33), (n_pts - 19, n_pts)):
        v, g = ctx.eval_nll_grad(th[a:b])
        assert np.array_equal(v, nll[a:b]) and np.array_equal(g, grad[a:b]), (a, b)
    ctx.close()


def test_more_analyses_than_one_launch_takes(monkeypatch):
    import paper_2607_00488_amd as nr
    monkeypatch.setenv("NR_GEMM_CONFIG", "0")
    ps = [inputs(40 + 9 * d, 20 + 31 * d, N_E, 50_000, 8320 + d, 8340 + d) for d in range(4)]
    ctxs, ths = [], []
    for d in range(19):
        ctxs.append(gpu_context(ps[d % 4]))
        ths.append(synth.theta_prior(1 + 7 * d, 8360 + d, f_range=(0.8, 1.2)))
    outs = nr.eval_nll_multi(ctxs, ths)
    for c, th, out in zip(ctxs, ths, outs):
        assert np.array_equal(out, c.eval_nll(th))
        c.close()
