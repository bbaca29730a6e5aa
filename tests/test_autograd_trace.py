"""The attention under torch.jit.trace, on the CPU: a dense stand-in for the two kernel calls, which like them is not
made of operators that a tracer sees."""
import numpy as np
import torch

import paper_2309_12578_amd as sp
from paper_2309_12578_amd import binding


def _probabilities(q, k):
    s = q.detach().numpy() @ k.detach().numpy().swapaxes(-1, -2) * 0.125
    lse = np.log(np.exp(s).sum(-1))
    return np.exp(s - lse[..., None]), lse


def _fwd(q, k, v, pattern, scale=0.0, flags=0, O=None):
    p, lse = _probabilities(q, k)
    O.numpy()[...] = p @ v.detach().numpy()
    return O, torch.from_numpy(lse)


def _bwd(q, k, v, o, do, lse, pattern, scale=0.0, flags=0):
    (p, _), (q, k, v, o, do) = _probabilities(q, k), [t.detach().numpy() for t in (q, k, v, o, do)]
    ds = p * (do @ v.swapaxes(-1, -2) - (do * o).sum(-1, keepdims=True)) * 0.125
    return tuple(torch.from_numpy(t) for t in (ds @ k, ds.swapaxes(-1, -2) @ q, p.swapaxes(-1, -2) @ do))


def _dense(q, k, v):
    return torch.softmax(q @ k.transpose(-1, -2) * 0.125, dim=-1) @ v


def test_trace_records_an_operator(monkeypatch):
    monkeypatch.setattr(binding, "attn_fwd", _fwd)
    monkeypatch.setattr(binding, "attn_bwd", _bwd)
    index = torch.zeros(2, dtype=torch.int32)
    pat = sp.Pattern(16, 16, index, index, index, index, index, index, index, index, 1)
    gen = torch.Generator().manual_seed(1)
    first, other = [[torch.randn((1, 2, 16, 64), generator=gen) for _ in range(3)] for _ in range(2)]
    for needs_grad in (False, True):
        for t in first + other:
            t.requires_grad_(needs_grad)
        traced = torch.jit.trace(lambda q, k, v: sp.sparse_attention(q, k, v, pat), first, check_trace=False)
        got, want = traced(*other), _dense(*other)
        assert torch.allclose(got, want, rtol=1e-5, atol=1e-6)
        if needs_grad:
            do = torch.randn(got.shape, generator=gen)
            for a, b in zip(torch.autograd.grad(got, other, do), torch.autograd.grad(want, other, do)):
                assert torch.allclose(a, b, rtol=1e-5, atol=1e-6)
