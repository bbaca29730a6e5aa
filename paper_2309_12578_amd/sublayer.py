"""The sparse multi-head-attention sub-layer of Algorithm 5 as a torch module.

Glue around the library: the four projections (hipBLASLt GEMMs but for the weight gradients), dropout and
the residual are torch ops; LayerNorm is the library's, and the head split and lines 4-7 of Algorithm 5
(SDDMM, sparse softmax, SpMM for every head) are one call into it, forward and backward.
"""
from __future__ import annotations

import torch
from torch import nn
from torch.nn.modules import module as _module

from . import binding as _b
from .autograd import sparse_attention

HEAD_DIM = 64   # the only head dimension the kernels are built for


class _Norm(nn.LayerNorm):
    """nn.LayerNorm by the library's kernels (csrc/norm_kernels.hip) where they take the call."""

    def forward(self, x: torch.Tensor) -> torch.Tensor:
        y = None
        if x.is_cuda and self.weight is not None and self.bias is not None and not torch.compiler.is_compiling():
            y = (_b._host or _b._native()).layer_norm(x, self.weight, self.bias, self.eps)
        return super().forward(x) if y is None else y


class _Projection(nn.Linear):
    """nn.Linear whose bf16 weight gradient, few outputs and a sum over every token, is a kernel of the
    library (csrc/projection_kernels.hip)."""

    def forward(self, x: torch.Tensor) -> torch.Tensor:
        y = None
        if x.is_cuda and not torch.compiler.is_compiling():
            y = (_b._host or _b._native()).projection(x, self.weight, self.bias)
        return super().forward(x) if y is None else y


def _hands_on(projection: nn.Module) -> bool:
    """Whether code other than _Projection's is handed the projection's input or output (a hook, another forward): it may
    change them in place, also where no version counter tells, while the attention beside it has saved them."""
    if getattr(type(projection), "forward", None) is not _Projection.forward:
        return True
    d = projection.__dict__
    return bool(d["_forward_pre_hooks"] or d["_forward_hooks"] or "forward" in d or
                _module._global_forward_pre_hooks or _module._global_forward_hooks)


class SparseMHA(nn.Module):
    """O = dropout(concat_h(sparse_attention(Q_h, K_h, V_h, P)) W^O) + E with
    Q, K, V = LayerNorm(E) W^{Q,K,V} (Algorithm 5).  `embed_dim` must be 64 * heads."""

    def __init__(self, embed_dim: int, heads: int, dropout: float = 0.0, bias: bool = False,
                 device=None, dtype=None):
        super().__init__()
        if embed_dim != heads * HEAD_DIM:
            raise ValueError("embed_dim must be %d * heads" % HEAD_DIM)
        kw = dict(device=device, dtype=dtype)
        self.heads = heads
        self.norm = _Norm(embed_dim, **kw)
        self.w_qkv = _Projection(embed_dim, 3 * embed_dim, bias=bias, **kw)   # W^Q | W^K | W^V
        self.w_o = _Projection(embed_dim, embed_dim, bias=bias, **kw)
        self.drop = nn.Dropout(dropout)

    def forward(self, E: torch.Tensor, pattern: _b.Pattern, flags: int = 0) -> torch.Tensor:
        """E: [B, L, embed_dim] on the GPU (bf16 or fp32); pattern: the layer's sparsity pattern."""
        B, L, D = E.shape
        w_qkv, w_o = self.w_qkv, self.w_o
        X = self.norm(E)
        qkv = w_qkv(X)
        S, R = None, E
        if qkv.is_cuda and not torch.compiler.is_compiling():
            R = (_b._host or _b._native()).residual(E, X)   # E, its gradient added up in LayerNorm's pass
            # lines 4-7 for every head, on the heads as they lie in qkv
            S = (_b._host or _b._native()).heads_attention(
                qkv, self.heads, pattern.row_ptr, pattern.col_idx, pattern.col_ptr, pattern.row_idx, pattern.bsr_pos,
                pattern.nnzb, pattern.block, flags, _hands_on(w_qkv) or _hands_on(w_o))
        if S is None:
            qkv = qkv.view(B, L, 3, self.heads, HEAD_DIM)
            # [B, H, L, 64] contiguous per tensor: the layout the kernels take
            Q, K, V = [qkv[:, :, i].transpose(1, 2).contiguous() for i in range(3)]
            S = sparse_attention(Q, K, V, pattern, flags=flags)               # lines 4-7, all heads at once
            S = S.transpose(1, 2).reshape(B, L, D)                            # concatenate the heads
        return self.drop(w_o(S)) + R
