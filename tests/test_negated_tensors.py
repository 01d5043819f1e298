"""Tensors whose stored values are not their values (torch's lazily negated
views): the calls that hand the library a pointer to a caller's tensor hand it
the values.  On the CPU, with the library's calls replaced by ones that read the
memory they are given."""
import ctypes
import types

import numpy as np
import torch

from paper_2607_00488_amd import autograd, surrogate


def at(ptr, shape, dtype):
    c = {np.float64: ctypes.c_double, np.float32: ctypes.c_float, np.int64: ctypes.c_int64}[dtype]
    return np.ctypeslib.as_array(ctypes.cast(ptr, ctypes.POINTER(c)), shape).copy()


def values(*shape):
    return torch.arange(1.0, 1.0 + np.prod(shape), dtype=torch.float64).reshape(shape)


def test_autograd_theta(monkeypatch):
    seen = []
    monkeypatch.setattr(torch.cuda, "current_stream", lambda dev=None: None)
    monkeypatch.setattr(autograd, "eval_nll_multi_dev", lambda c, th, nll, grad, stream:
                        seen.append(at(th[0].data_ptr(), tuple(th[0].shape), np.float64)))
    theta = torch._neg_view(values(3, 7))
    assert theta.is_contiguous() and theta.is_neg()
    autograd.nll(theta, types.SimpleNamespace(n_theta=7))
    assert np.array_equal(seen[0], -values(3, 7).numpy())


def test_training_tensors(monkeypatch):
    rows = []

    def step(h, th, tg, B, lr, want, stream):
        rows.append((at(th, (B, 7), np.float64), at(tg, (B, 16), np.float32)))

    def epoch(h, th, tg, idx, n, B, lr, stream):
        i = at(idx, (n, B), np.int64)
        t, g = at(th, (16, 7), np.float64), at(tg, (16, 16), np.float32)
        rows.extend((t[k], g[k]) for k in i)

    s = types.SimpleNamespace
    monkeypatch.setattr(torch.cuda, "current_stream", lambda dev=None: s(cuda_stream=0))
    monkeypatch.setattr(torch.cuda, "synchronize", lambda dev=None: None)
    monkeypatch.setattr(surrogate, "nr_mlp_train_step_dev", step)
    monkeypatch.setattr(surrogate, "nr_mlp_train_epoch_dev", epoch)
    net = s(dev=torch.device("cpu"), h=None, hidden=256, n_out=16)
    theta, targets = values(16, 7), values(16, 16).float()
    out = []
    for t, g in ((theta, targets), (torch._neg_view(-theta), targets),
                 (theta, torch._neg_view(-targets))):
        rows.clear()
        surrogate.Surrogate.train(net, t, g, epochs=1, batch=8, seed=3)
        out.append([np.concatenate([a.ravel() for a in r]) for r in rows])
    assert np.array_equal(out[1], out[0]) and np.array_equal(out[2], out[0])
