"""Calls whose route through the kernels is picked on the host by shape, option
or list, each against the FP64 oracle or a call by another route."""
import numpy as np
import pytest

import synth
from problems import gpu_context, inputs

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -53


def log(msg):
    print("[gpu]", msg, flush=True)


@pytest.mark.parametrize("points", [(5, 40, 17), (5, 600, 17)])
def test_grouped_call_with_a_context_several_times(points, monkeypatch):
    """Every entry's results are those of its own call: with the split pinned
    the same sums, bit for bit."""
    import torch
    import paper_2607_00488_amd as nr
    monkeypatch.setenv("NR_GEMM_CONFIG", "0")
    a = gpu_context(inputs(96, 129, 24, 100_000, 8501, 8502))
    b = gpu_context(inputs(40, 70, 24, 100_000, 8503, 8504))
    ctxs = [a, b, a]
    ths = [synth.theta_prior(n, 8505 + i, f_range=(0.8, 1.2)) for i, n in enumerate(points)]
    log(f"grouped call, one context twice, {points} points")
    ref = [c.eval_nll_grad(t) for c, t in zip(ctxs, ths)]
    for v, (r, _) in zip(nr.eval_nll_multi(ctxs, ths), ref):
        assert np.array_equal(v, r)
    tt = [torch.tensor(t, device="cuda:0") for t in ths]
    nll = [torch.empty(len(t), dtype=torch.float64, device="cuda:0") for t in ths]
    grad = [torch.empty(len(t), 7, dtype=torch.float64, device="cuda:0") for t in ths]
    nr.eval_nll_multi_dev(ctxs, tt, nll, grad)
    torch.cuda.synchronize()
    for v, g, (r, s) in zip(nll, grad, ref):
        assert np.array_equal(v.cpu().numpy(), r) and np.array_equal(g.cpu().numpy(), s)
    a.close()
    b.close()


@pytest.mark.parametrize("n_t,n_reco,points", [
    (130, 77, (3, 16, 17, 33, 49, 65, 113)), (1000, 33, (5, 129)), (31, 2, (3, 18)),
    (700, 4100, (3, 500))])
def test_blocks_of_a_multi_component_list(n_t, n_reco, points, monkeypatch):
    """Lists of three or more points of a multi-component context (blocked fold)
    against its points one at a time (the single-point launches): block and group
    edges in the points, ragged rows and columns, more row splits than a round of
    loads, and a list that takes the workspace several times.

    Tolerance: the two routes add the same products in different orders and form
    the weights from suffix sums or from the recoil basis, so a mu_j carries at
    most (rows + nodes + 128) roundings of 2^-53 relative, and -2lnL moves by
    2 sum_j |mu_j - n_j| times that plus its own summation."""
    import paper_2607_00488_amd as nr
    k = synth.component_inputs(n_t, n_reco, 200_000, 8521)
    args = [k.pop(n) for n in ("comp_of_source", "hist", "scale", "rate_sm")]
    ctx = nr.Context(0)
    ctx.set_sources(synth.source_nodes(48), n_t)
    ctx.set_components(*args, **k)
    g = synth.rng(8522)
    th = g.uniform(0.8, 1.2, (max(points), ctx.n_theta))
    th[:, :5] = synth.theta_prior(len(th), 8523)[:, :5]
    ctx.set_data(np.ones(n_reco), None)
    n = g.poisson(ctx.eval_mu(th[:1])[0]).astype(np.float64)
    ctx.set_data(n, None)
    log(f"blocks, {n_t} x {n_reco}, {points} points")
    one = sorted({0, 1, 2, *(i for p in points for i in (p // 2, p - 1))})
    mu = {i: ctx.eval_mu(th[i:i + 1])[0] for i in one}
    nll = {i: ctx.eval_nll(th[i:i + 1])[0] for i in one}
    rel = (5 * n_t + 3 * 48 + 2 + 128) * EPS
    full = ctx.eval_nll(th)
    for p in points:
        got, gmu = ctx.eval_nll(th[:p]), ctx.eval_mu(th[:p])
        assert np.array_equal(got, full[:p]), p  # whatever list a point is in
        for i in one:
            if i >= p:
                continue
            assert np.all(np.abs(gmu[i] - mu[i]) <= rel * np.abs(mu[i])), (p, i)
            tol = 2 * np.abs(mu[i] - n).sum() * rel + 2 * (mu[i] + n).sum() * 64 * EPS
            assert abs(got[i] - nll[i]) <= tol, (p, i)
    ctx.close()


def diagonal(n_t, n_reco, width, seed):
    """An analysis whose response rows are non-zero over `width` bins only."""
    import paper_2607_00488_amd as nr
    g = synth.rng(seed)
    c = np.arange(n_t) * n_reco // n_t
    j = np.arange(n_reco)
    R = np.where(np.abs(j - c[:, None]) <= width // 2,
                 g.uniform(0.5, 1.5, (n_t, n_reco)), 0.0).astype(np.float32)
    ctx = nr.Context(0)
    ctx.set_sources(synth.source_nodes(24), n_t)
    ctx.set_response(R, n_sig=1.0e4)
    b = np.full(n_reco, 10.0)
    ctx.set_data(b, b)
    n = g.poisson(ctx.eval_mu(synth.theta_sm()[None])[0]).astype(np.float64)
    ctx.set_data(n, b)
    return ctx


@pytest.mark.parametrize("n_t,n_reco,width", [
    (4096, 2048, 100), (1003, 777, 60), (129, 1025, 30), (700, 321, 9), (2050, 1153, 450)])
def test_bands_narrow_and_wide(n_t, n_reco, width, monkeypatch):
    """Band skipping on responses whose bands are narrow (tiles of 64 columns) and
    wide: every entry point bit for bit as without, also beside an analysis without
    bands in one grouped call."""
    import torch
    import paper_2607_00488_amd as nr
    monkeypatch.setenv("NR_GEMM_CONFIG", "0")
    ctx, other = diagonal(n_t, n_reco, width, 8531), diagonal(100, 300, 300, 8532)
    th = synth.theta_prior(19, 8533, f_range=(0.8, 1.2))
    log(f"bands, {n_t} x {n_reco}, {width} bins wide")

    def values():
        dev = [torch.tensor(t, device="cuda:0") for t in (th, th[:7], th[3:])]
        nll = [torch.empty(len(t), dtype=torch.float64, device="cuda:0") for t in dev]
        nr.eval_nll_multi_dev([ctx, other, ctx], dev, nll)
        torch.cuda.synchronize()
        ctx.build_templates()
        return [ctx.eval_nll(th), ctx.eval_nll(th[:1]), *ctx.eval_nll_grad(th), ctx.eval_mu(th),
                ctx.eval_nll_batched(th), *ctx.eval_nll_grad_batched(th[:3]),
                *ctx.eval_nll_templates(th, grad=True), *(v.cpu().numpy() for v in nll)]

    dense = values()
    ctx.set_band_skipping(True)
    for i, (a, b) in enumerate(zip(dense, values())):
        assert np.array_equal(a, b), i
    ctx.close()
    other.close()


@pytest.mark.parametrize("n_t,n_reco", [
    (1100, 34001), (1024, 39936), (1030, 41003), (1025, 23001), (301, 34001), (40, 8193),
    (5001, 20), (16384, 65)])
def test_row_splits_of_wide_and_of_tall_responses(n_t, n_reco):
    """Responses whose rows the fold splits by another rule than their size: many
    columns (four waves over the same 64, one split and two) and few (fewer splits
    than compute units); band skipping and the allocation-free call bit for bit.

    Tolerances of the basis form's other edges (tests/test_gpu_shared.py): rel =
    (rows + nodes + 128) roundings of a mu_j, and what they and its own summation
    move -2lnL and the gradient by.  -2lnL is compared as the difference of two
    points with the exactly rounded sum over the oracle's spectra: the data constant,
    and the oracle's own -2lnL, are sums of all bins in a row, whose rounding at
    40000 bins is as large as the tolerance."""
    import math
    import torch
    N_E = 24
    p = inputs(n_t, n_reco, N_E, 400_000, 8541, 8542)
    ctx = gpu_context(p)
    th = synth.theta_prior(18, 8543, f_range=(0.8, 1.2))
    log(f"row splits, {n_t} x {n_reco}")
    nll, grad = ctx.eval_nll_grad(th)
    o, n, mu = p["oracle"], p["n"], ctx.eval_mu(th)
    rel = (n_t + 3 * N_E + 2 + 128) * EPS
    ref, tol = {}, {}
    for i in (0, 17):
        m, g = o.mu(th[i]), o.nll_grad(th[i])[1]
        assert np.all(np.abs(mu[i] - m) <= rel * np.abs(m)), i
        ref[i] = 2 * math.fsum([*m, *(-k * math.log(x) for k, x in zip(n, m) if k > 0)])
        tol[i] = 2 * np.abs(m - n).sum() * rel + 2 * (m + n).sum() * 64 * EPS
        w = np.abs(2 * (1 - n / m)) + 2 * n / m
        for k in range(7):
            d = np.zeros_like(m)
            for s in (-1.0, 1.0):
                t = th[i].copy()
                t[k] += s
                d += np.abs(o.mu(t) - m)
            assert abs(grad[i, k] - g[k]) <= 8 * rel * (w * d).sum(), (i, k)
    assert abs(nll[17] - nll[0] - (ref[17] - ref[0])) <= tol[0] + tol[17]
    for i in (1, 2, 3):  # one and two points add many slices another way
        assert np.array_equal(ctx.eval_nll(th[-i:]), nll[-i:])
    tt = torch.tensor(th, device="cuda:0")
    out = torch.empty(len(th), dtype=torch.float64, device="cuda:0")
    ctx.eval_nll_dev_noalloc(tt, out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), nll)
    ctx.set_band_skipping(True)
    assert np.array_equal(ctx.eval_nll(th), nll)
    ctx.close()


@pytest.mark.parametrize("n_t,n_reco", [(75_001, 1001), (2300, 34001)])
def test_responses_beyond_the_cache(n_t, n_reco):
    """Responses that are read past the caches, in rows padded to whole lines (300 MB
    and more), of ragged sizes: spectra against the sums of the rows with the weights
    of the single-point launches, likelihood and gradient against the spectra."""
    import paper_2607_00488_amd as nr
    g = synth.rng(8551)
    R = g.random((n_t, n_reco), dtype=np.float32) / np.float32(n_reco)
    n, b = g.poisson(20.0, n_reco).astype(np.float64), np.full(n_reco, 10.0)
    m = g.uniform(0.5, 1.5, n_t) * 1.0e4 / n_t
    src = synth.source_nodes(8)
    th = synth.theta_prior(3, 8552, f_range=(0.8, 1.2))

    log(f"beyond the cache, {n_t} x {n_reco}")
    ctx = nr.Context(0)
    ctx.set_sources(src, n_t)
    ctx.set_response(R, m=m)
    ctx.set_data(n, b)
    mu = ctx.eval_mu(th)
    nll, grad = ctx.eval_nll_grad(th)
    w = ctx.eval_weights(th)
    ref = th[:, 6:] * b + np.array([(m * x) @ R.astype(np.float64) for x in w])
    rel = (n_t + 3 * 8 + 2 + 128) * EPS
    assert np.all(np.abs(mu - ref) <= rel * ref)
    one = 2 * (mu - n * np.log(mu)).sum(1)
    tol = 2 * np.abs(mu - n).sum(1) * rel + 2 * (mu + n).sum(1) * 64 * EPS
    assert abs((nll[1] - nll[0]) - (one[1] - one[0])) <= tol[0] + tol[1]
    # mu is linear in f_bkg and f_8B: exact differences
    a = 2 * (1 - n / mu)
    for k in (5, 6):
        up = th.copy()
        up[:, k] += 1.0
        d = ctx.eval_mu(up) - mu
        bound = 8 * rel * ((np.abs(a) + 2 * n / mu) * (np.abs(d) + 2 * mu)).sum(1)
        assert np.all(np.abs(grad[:, k] - (a * d).sum(1)) <= bound), k
    assert np.array_equal(ctx.eval_nll(th[:1]), nll[:1])
    ctx.set_band_skipping(True)
    assert np.array_equal(ctx.eval_nll(th), nll)
    ctx.close()


@pytest.mark.parametrize("B", [0, 1, 4, 5])
def test_one_component_in_the_template_form(B):
    """The smallest column class (one component and up to four backgrounds, the
    first count beyond it) at sizes off the tiles, with the tolerances and the exact
    differences of tests/test_gpu_shared.py."""
    from test_gpu_shared import test_multi_component_columns
    log(f"one component, {B} backgrounds")
    test_multi_component_columns(1, B)


def test_point_by_point_route_and_its_adjoint():
    """A single-component response of so many bins that the basis form does not fit
    the allocation-free workspace: the single-point launches and the adjoint of the
    fold.  Likelihood and gradient with pulls against the oracle, band skipping, the
    allocation-free call and a replayed graph bit for bit, the batched (basis) form
    as another route.  Tolerances as above; the pulls are a few exact operations."""
    import math
    import torch
    n_t, n_reco, N_E = 40, 60001, 24
    p = inputs(n_t, n_reco, N_E, 400_000, 8561, 8562)
    mean = np.array([0.1, 0, 0, 0, 2.0, 1.0, 1.0])
    sigma = np.array([0.5, 0, 0, 0, 3.0, 0.1, 0.1])
    ctx = gpu_context(p, pulls=(mean, sigma))
    th = synth.theta_prior(5, 8563, f_range=(0.8, 1.2))
    log(f"point by point, {n_t} x {n_reco}")
    on = sigma > 0
    pull = (((th - mean)[:, on] / sigma[on]) ** 2).sum(1)
    dpull = np.where(on, 2 * (th - mean) / np.where(on, sigma, 1.0) ** 2, 0.0)
    nll, grad = ctx.eval_nll_grad(th)
    mu = ctx.eval_mu(th)
    o, n = p["oracle"], p["n"]
    rel = (n_t + 3 * N_E + 2 + 128) * EPS
    ref, tol, w = np.zeros(5), np.zeros(5), np.zeros((5, n_reco))
    for i in range(5):
        m, g = o.mu(th[i]), o.nll_grad(th[i])[1]
        assert np.all(np.abs(mu[i] - m) <= rel * np.abs(m)), i
        ref[i] = 2 * math.fsum([*m, *(-k * math.log(x) for k, x in zip(n, m) if k > 0)]) + pull[i]
        tol[i] = 2 * np.abs(m - n).sum() * rel + 2 * (m + n).sum() * 64 * EPS
        w[i] = np.abs(2 * (1 - n / m)) + 2 * n / m
        for k in range(7):
            d = np.zeros_like(m)
            for s in (-1.0, 1.0):
                t = th[i].copy()
                t[k] += s
                d += np.abs(o.mu(t) - m)
            assert abs(grad[i, k] - g[k] - dpull[i, k]) <= \
                8 * rel * (w[i] * d).sum() + 8 * EPS * abs(dpull[i, k]), (i, k)
    assert np.all(np.abs(nll - nll[0] - (ref - ref[0])) <= tol + tol[0])
    # another route: the grouped calls take the basis form
    bn, bg = ctx.eval_nll_grad_batched(th)
    assert np.all(np.abs(bn - nll) <= 2 * tol)
    tt = torch.tensor(th, device="cuda:0")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    for call in (ctx.eval_nll_dev, ctx.eval_nll_dev, ctx.eval_nll_dev_noalloc):
        out = torch.full((5,), float("nan"), dtype=torch.float64, device="cuda:0")
        g = torch.full((5, 7), float("nan"), dtype=torch.float64, device="cuda:0")
        torch.cuda.synchronize()
        for _ in range(3):  # the second and third replay the first's graph
            call(tt, out, g, stream=s)
            s.synchronize()
            assert np.array_equal(out.cpu().numpy(), nll)
            assert np.array_equal(g.cpu().numpy(), grad)
        call(tt, out, stream=s)
        s.synchronize()
        assert np.array_equal(out.cpu().numpy(), ctx.eval_nll(th))
    plain = ctx.eval_nll(th)
    assert np.all(np.abs(plain - nll) <= 2 * tol)
    ctx.set_band_skipping(True)
    v, g = ctx.eval_nll_grad(th)
    assert np.array_equal(v, nll) and np.array_equal(g, grad)
    assert np.array_equal(ctx.eval_nll(th), plain)
    ctx.close()


@pytest.mark.parametrize("B,N", [(136, 1096), (72, 1608), (264, 4008)])
def test_training_steps_of_either_gradient_tile(B, N):
    """The last counts of outputs with 64 x 32 tiles of the weight gradient and ones
    with 64 x 96, ragged, through the checks of the smaller networks."""
    from test_gpu_train import test_ragged_steps
    log(f"training step, {B} points x {N} outputs")
    test_ragged_steps(B, N)
