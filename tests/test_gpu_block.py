"""The blocked fold (lists of three or more points share the stream over R)
against the single-point launches, other kernels, point by point: block and
group edges in the number of points, ragged rows and columns, the stacked
multi-component rows, band skipping, and lists longer than one workspace.

Tolerance: the two routes add the same products in different orders, and form
the weights from a table of suffix sums or from the recoil basis, so a mu_j
carries at most (rows + nodes + 128) roundings of 2^-53 relative; -2lnL then
moves by 2 sum_j |mu_j - n_j| times that, plus its own summation."""
import numpy as np
import pytest

import synth
from problems import gpu_context, inputs

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -53


def singles(ctx, th):
    nll = np.array([ctx.eval_nll(t[None])[0] for t in th])
    mu = np.vstack([ctx.eval_mu(t[None]) for t in th])
    return nll, mu


def check(ctx, th, n, n_rows, n_nodes, what):
    nll, mu = singles(ctx, th)
    got, gmu = ctx.eval_nll(th), ctx.eval_mu(th)
    rel = (n_rows + n_nodes + 128) * EPS
    assert np.all(np.abs(gmu - mu) <= rel * np.abs(mu)), what
    tol = 2.0 * np.abs(mu - n).sum(1) * rel + 2.0 * (mu + n).sum(1) * 64 * EPS
    assert np.all(np.abs(got - nll) <= tol), (what, np.max(np.abs(got - nll) / tol))


@pytest.mark.parametrize("n_t,n_reco,n_pts", [
    (7, 3, 3), (64, 5, 16), (333, 77, 17), (97, 257, 33), (1000, 1023, 49),
    (2100, 300, 65), (512, 256, 113)])
def test_blocks_match_single_points(n_t, n_reco, n_pts):
    p = inputs(n_t, n_reco, 37, 200_000, 8100 + n_t, 8101 + n_t)
    ctx = gpu_context(p)
    th = synth.theta_prior(n_pts, 8102, f_range=(0.8, 1.2))
    check(ctx, th, p["n"], n_t, 3 * 37 + 2, (n_t, n_reco, n_pts))
    ctx.close()


def test_a_points_result_does_not_depend_on_its_list():
    """Bitwise: alone in a list of three, or anywhere in a longer one, and in
    the allocation-free entry point, whose workspace holds fewer points."""
    import torch
    p = inputs(4096, 2048, 64, 400_000, 8111, 8112)
    ctx = gpu_context(p)
    th = synth.theta_prior(300, 8113, f_range=(0.8, 1.2))
    full = ctx.eval_nll(th)
    for a, b in ((0, 3), (17, 40), (250, 300)):
        assert np.array_equal(ctx.eval_nll(th[a:b]), full[a:b]), (a, b)
    dev = torch.device("cuda:0")
    tt = torch.tensor(th, dtype=torch.float64, device=dev)
    out = torch.empty(300, dtype=torch.float64, device=dev)
    ctx.eval_nll_dev_noalloc(tt, out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), full)
    ctx.close()


@pytest.mark.parametrize("n_t,n_reco", [(130, 77), (512, 256)])
def test_blocks_multi_component(n_t, n_reco):
    import paper_2607_00488_amd as nr
    k = synth.component_inputs(n_t, n_reco, 200_000, 8121)
    ctx = nr.Context(0)
    ctx.set_sources(synth.source_nodes(48), n_t)
    ctx.set_components(k.pop("comp_of_source"), k.pop("hist"), k.pop("scale"),
                       k.pop("rate_sm"), **k)
    g = synth.rng(8122)
    th = g.uniform(0.8, 1.2, (19, ctx.n_theta))
    th[:, :5] = synth.theta_prior(19, 8123)[:, :5]
    ctx.set_data(np.ones(n_reco), None)
    n = g.poisson(ctx.eval_mu(th[:1])[0]).astype(np.float64)
    ctx.set_data(n, None)
    check(ctx, th, n, 5 * n_t, 48 * 3 + 2, (n_t, n_reco))
    for on in (True, False):
        ctx.set_band_skipping(on)
        v = ctx.eval_nll(th)
        assert on or np.array_equal(v, band)
        band = v
    ctx.close()
