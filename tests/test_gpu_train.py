"""The fused training step (hidden layers of 256) at ragged batches and outputs:
its gradients against the numpy reference with the same weights, block by block,
at the edges of the 32-point chains, the 128 x 128 output tiles, the
64 x 96 gradient tiles and the chunks of the reductions; then Adam, from the
step's own gradients; then a second step, whose reference takes the updated
weights, so that every copy of them the step keeps is seen to follow.

Gradient tolerance: both sides round the same quantities to BF16, but a sum that
lands beside a rounding boundary may fall on either neighbour, 2^-7 apart
relative, in each of the two operands of a product and at each of the four
layers behind it.  Were all of them off, with independent signs, the difference
would be sqrt(8) 2^-7 of the gradient in the 2-norm: 2^-5 with margin, held by
every layer as a whole and by every block of 32 of its outputs and of its inputs,
so that a tile, a chunk of a reduction or an edge left out (the smallest, 8 of
2056 points, changes a norm by 6 %) shows.  Adam is ten FP32 operations on the
same FP32 inputs: 16 roundings of the update and of w."""
import numpy as np
import pytest

import synth
from oracle import mlp as ref

pytestmark = pytest.mark.gpu

H = 256


@pytest.mark.parametrize("B,N", [(8, 8), (40, 136), (72, 64), (200, 72), (136, 1000), (2056, 264)])
def test_ragged_steps(B, N):
    import torch
    from paper_2607_00488_amd import nr_mlp_set_output_norm, nr_mlp_train_step_dev
    from paper_2607_00488_amd.surrogate import Surrogate, init_params
    lo, hi = synth.theta_box()
    s = Surrogate(N, lo, hi, hidden=H, seed=21)
    params = init_params(H, N, 22, out_scale=1.0)
    s.set_params(params)
    nr_mlp_set_output_norm(s.h, np.zeros(N, np.float32), np.ones(N, np.float32))
    g = synth.rng(23 + B)
    th = g.uniform(lo, hi, (B, 7))
    tg = g.standard_normal((B, N)).astype(np.float32)
    tt = torch.tensor(th, device="cuda:0")
    tgt = torch.tensor(tg, device="cuda:0")
    m = np.zeros(len(params))
    v = np.zeros(len(params))
    lr, b1, b2, eps = (float(np.float32(x)) for x in (1e-3, 0.9, 0.999, 1e-8))
    for step in (1, 2):
        loss = nr_mlp_train_step_dev(s.h, tt.data_ptr(), tgt.data_ptr(), B, lr, True)
        got = s.grads().astype(np.float64)
        rl, rg = ref.mse_grad(params.astype(np.float64), th, tg.astype(np.float64), lo, hi, H, N,
                              bf16=True)
        o = 0
        for rows, kp, kin in ((H, 32, 7), (H, H + 8, H), (H, H + 8, H), (N, H + 8, H)):
            a, b = (x[o:o + rows * kp].reshape(rows, kp) for x in (got, rg))
            o += rows * kp
            assert np.all(a[:, kin + 1:] == 0.0)
            parts = ([(a[r:r + 32], b[r:r + 32]) for r in range(0, rows, 32)] +
                     [(a[:, c:c + 32], b[:, c:c + 32]) for c in range(0, kin + 1, 32)])
            for x, y in [(a, b)] + parts:
                assert np.linalg.norm(x - y) <= 2.0 ** -5 * np.linalg.norm(y), (step, rows, kp)
        assert loss == pytest.approx(rl, rel=1e-4)
        m = b1 * m + (1 - b1) * got
        v = b2 * v + (1 - b2) * got ** 2
        up = lr * (m / (1 - b1 ** step)) / (np.sqrt(v / (1 - b2 ** step)) + eps)
        new = s.params()
        want = params.astype(np.float64) - up
        # bc2 = 1 - b2^t is formed in FP32 from a number beside one: 2^-24 / 1e-3
        tol = 2.0 ** -20 * np.abs(want) + (2.0 ** -20 + 2.0 ** -24 / (1 - b2)) * np.abs(up)
        assert np.all(np.abs(new - want) <= tol), (step, np.max(np.abs(new - want) / tol))
        params = new
    s.close()


@pytest.mark.parametrize("P,batch,N", [(1000, 136, 72), (4096, 2048, 264), (50, 64, 8)])
def test_gathered_epochs_match_stepwise_training(P, batch, N):
    """Whole epochs whose kernels gather the batches, against the same epochs step
    by step on tensors gathered before (asking for losses selects that): bitwise,
    a batch larger than the sample (no step at all) included."""
    import torch
    from paper_2607_00488_amd.surrogate import Surrogate
    lo, hi = synth.theta_box()
    g = synth.rng(31)
    th = torch.tensor(g.uniform(lo, hi, (P, 7)), device="cuda:0")
    tg = torch.tensor(g.standard_normal((P, N)).astype(np.float32), device="cuda:0")
    out = []
    for log_every in (0, 1):
        s = Surrogate(N, lo, hi, hidden=H, seed=32)
        r = s.train(th, tg, epochs=3, batch=batch, log_every=log_every)
        assert r["steps"] == 3 * (P // batch)
        out.append(s.params())
        s.close()
    assert np.array_equal(*out)
