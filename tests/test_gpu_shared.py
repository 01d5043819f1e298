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
    p = inputs(64, 256, N_E, 100_000, 8311, 8312)
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


@pytest.mark.parametrize("K,B", [(1, 0), (5, 4), (4, 8), (5, 5), (8, 8)])
def test_multi_component_columns(K, B):
    """Both column classes, their last columns and the padded bins, against the
    streaming path (other kernels): spectra and likelihoods directly, the
    gradient from its spectra, which are quadratic in the couplings and linear
    in m2 and the rates, so that a central difference over a unit step is exact."""
    import paper_2607_00488_amd as nr
    n_t, n_reco, P = 67, 33, 21
    src = (synth.source_nodes(N_E) * 2)[:max(K, 5)]
    g = synth.rng(8400 + 10 * K + B)
    shapes = [(16.0, 2.0 + k) for k in range(K)]
    d = synth.component_inputs(n_t, n_reco, 30_000, 8401, shapes=shapes)
    ctx = nr.Context(0)
    ctx.set_sources(src, n_t)
    ctx.set_components(np.arange(len(src), dtype=np.int32) % K, d["hist"],
                       g.uniform(0.8, 1.2, K), g.uniform(50.0, 500.0, K),
                       bkg_pdf=g.uniform(0.5, 1.5, (B, n_reco)) / n_reco if B else None,
                       bkg_rate=g.uniform(50.0, 500.0, B) if B else None,
                       comp_mask=d["comp_mask"], mask=d["mask"], exposure=1.5)
    th = g.uniform(0.8, 1.2, (P, 5 + K + B))
    th[:, :5] = synth.theta_prior(P, 8402)[:, :5]
    ctx.set_data(np.ones(n_reco), None)
    n = g.poisson(ctx.eval_mu(th[:1])[0]).astype(np.float64)
    ctx.set_data(n, None)
    rel = (n_t + 3 * N_E + 2 + 128) * EPS
    mu, nll = ctx.eval_mu(th), ctx.eval_nll(th)
    assert np.all(np.abs(ctx.eval_mu_templates(th) - mu) <= rel * np.abs(mu))
    v, grad = ctx.eval_nll_templates(th, grad=True)
    tol = 2 * np.abs(mu - n).sum(1) * rel + 2 * (mu + n).sum(1) * 64 * EPS
    assert np.all(np.abs(v - nll) <= tol)
    assert np.array_equal(ctx.eval_nll_templates(th), v)
    q = np.divide(n, mu, out=np.zeros_like(mu), where=n > 0)  # an empty bin's a is 2
    a, w = 2 * (1 - q), np.abs(2 * (1 - q)) + 2 * q
    for k in range(5 + K + B):
        up, dn = th.copy(), th.copy()
        up[:, k] += 1.0
        dn[:, k] -= 1.0
        hi, lo = ctx.eval_mu(up) - mu, ctx.eval_mu(dn) - mu
        ref = (a * (hi - lo) / 2).sum(1)
        bound = 8 * rel * (w * (np.abs(hi) + np.abs(lo) + 2 * mu)).sum(1)
        assert np.all(np.abs(grad[:, k] - ref) <= bound), k
    ctx.close()
