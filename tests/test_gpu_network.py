"""The network's likelihood kernel where it takes theta in and hands -2lnL out itself:
one group of bins per point (up to 128 bins) against several (136), the first and
last rows of its 128-point tiles, pulls, and points outside the box.  Reference: the
network's own FP32 ln mu, summed in FP64 on the host.  The kernel's FP32 exponential
and its sums of four move mu_j by at most 1.25 2^-24 |ln mu_j| + 2^-23 + 3 2^-24
relative (2^-22 |ln mu_j| + 2^-20 with margin); the pulls are FP64 on both sides."""
import math

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [8, 128, 136])
@pytest.mark.parametrize("B", [8, 128, 136, 264])
def test_input_and_pulls(B, N):
    import torch
    import paper_2607_00488_amd as nr
    from paper_2607_00488_amd.surrogate import Surrogate, init_params
    g = synth.rng(31 + N)
    lo, hi = synth.theta_box()
    n = g.poisson(5.0, N).astype(np.float64)
    pm, ps = g.uniform(lo, hi), np.where(np.arange(7) % 3 == 1, 0.0, 0.3)
    ctx = nr.Context(0)
    ctx.set_sources(synth.source_nodes(64), 64)
    ctx.set_response((g.random((64, N)) / N).astype(np.float32), n_sig=1e4)
    ctx.set_data(n, np.full(N, 10.0), pm, ps)
    s = Surrogate(N, lo, hi, hidden=256, seed=32)
    s.set_params(init_params(256, N, 33, out_scale=1.0))
    nr.nr_mlp_set_output_norm(s.h, np.full(N, 1.5, np.float32), np.full(N, 0.3, np.float32))
    th = g.uniform(lo, hi, (B, 7))
    out = np.zeros(B, bool)
    for p, i, edge in ((0, 0, lo), (3, 6, hi), (B - 1, 4, hi)):
        th[p, i] = edge[i] + (0.25 if edge is hi else -0.25) * (hi[i] - lo[i])
        out[p] = True
    th[1] = lo  # on the edge: inside
    t = torch.tensor(th, device="cuda:0")
    got, outside = s.nll(ctx, t)
    lm = s.logmu(t).cpu().numpy().astype(np.float64)
    z = (th[:, ps > 0] - pm[ps > 0]) / ps[ps > 0]
    mu = np.exp(lm)
    ref = 2.0 * np.sum(mu - n * lm + [math.lgamma(x + 1.0) for x in n], axis=1) + np.sum(z * z, axis=1)
    bound = 2.0 * np.sum(mu * (np.abs(lm) * 2.0 ** -22 + 2.0 ** -20), axis=1)
    assert np.array_equal(outside.cpu().numpy() != 0, out)
    assert np.all(np.abs(got.cpu().numpy() - ref) <= bound + 1e-12 * np.abs(ref))
    s.close()
    ctx.close()
