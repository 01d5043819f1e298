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
