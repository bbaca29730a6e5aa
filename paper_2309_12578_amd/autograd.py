"""torch.autograd front end of the sparse attention (Section 4.3, "Integration of GPU kernels with
PyTorch": the shared library is loaded once and a custom autograd function calls its forward and
backward entry points).  Glue only: the autograd node is native (csrc/host_ext.cpp), under torch.jit.trace a
Python function that the tracer records, and both directions run in libspion's kernels."""
from __future__ import annotations

import torch

from . import binding as _b


class _TracedAttention(torch.autograd.Function):
    """The same calls as the native node, as an operator of a traced graph."""

    @staticmethod
    def forward(ctx, Q, K, V, pattern, scale, flags):
        Q, K, V = Q.contiguous(), K.contiguous(), V.contiguous()
        O = torch.empty_like(Q)   # the tracer asks for a tensor that an operator of torch made
        O, LSE = _b.attn_fwd(Q, K, V, pattern, scale=scale, flags=flags, O=O)
        ctx.save_for_backward(Q, K, V, O, LSE)
        ctx.pattern, ctx.scale, ctx.flags = pattern, scale, flags
        return O

    @staticmethod
    def backward(ctx, dO):
        Q, K, V, O, LSE = ctx.saved_tensors
        return *_b.attn_bwd(Q, K, V, O, dO.contiguous(), LSE, ctx.pattern, scale=ctx.scale, flags=ctx.flags), None, None, None


def sparse_attention(Q: torch.Tensor, K: torch.Tensor, V: torch.Tensor, pattern: _b.Pattern,
                     scale: float = 0.0, flags: int = 0) -> torch.Tensor:
    """Eq. 5 on the kept blocks of `pattern` for Q, K, V of shape [B, H, L, 64] (bf16 or fp32);
    differentiable with respect to Q, K and V."""
    O = (_b._host or _b._native()).sparse_attention(
        Q, K, V, pattern.row_ptr, pattern.col_idx, pattern.col_ptr, pattern.row_idx, pattern.bsr_pos, pattern.nnzb,
        pattern.block, scale, flags)
    return _TracedAttention.apply(Q, K, V, pattern, scale, flags) if O is None else O
