"""torch.autograd front end of the sparse attention (Section 4.3, "Integration of GPU kernels with
PyTorch": the shared library is loaded once and a custom autograd function calls its forward and
backward entry points).  Glue only: the autograd node is native (csrc/host_ext.cpp) and both directions
run in libspion's kernels."""
from __future__ import annotations

import torch

from . import binding as _b


def sparse_attention(Q: torch.Tensor, K: torch.Tensor, V: torch.Tensor, pattern: _b.Pattern,
                     scale: float = 0.0, flags: int = 0) -> torch.Tensor:
    """Eq. 5 on the kept blocks of `pattern` for Q, K, V of shape [B, H, L, 64] (bf16 or fp32);
    differentiable with respect to Q, K and V."""
    return (_b._host or _b._native()).sparse_attention(
        Q, K, V, pattern.row_ptr, pattern.col_idx, pattern.col_ptr, pattern.row_idx, pattern.bsr_pos, pattern.nnzb,
        pattern.block, scale, flags)
