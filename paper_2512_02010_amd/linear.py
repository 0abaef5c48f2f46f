"""The NVFP4 linear layer of Fig. 3 as a sequence of library calls.

Nothing is computed here: every function strings together ``nvfp4_46_scale_quantize`` (tensor
scale and codes from one call) and ``nvfp4_46_gemm`` the way the figure wires them.

    FPROP   y  = x W^T          x [T][K] BF16 rowwise, RTN          W [N][K] FP32 rowwise
    DGRAD   dx = dy W           dy [T][N] BF16 rowwise, SR          W columnwise (= W^T rowwise)
    WGRAD   dW = dy^T x         dy columnwise, Hadamard + SR        x columnwise, Hadamard

Every operand is quantized along the contraction axis of the product it enters.  The weight
matrix is quantized once per step, by default in 16x16 tiles (Section 4.1), which yields the
packing for W and for W^T with identical codes and scales.  Stochastic rounding is used on
the gradient operands, the random Hadamard transform on both operands of WGRAD (same sign
vector along the contraction axis, so it cancels in the product).

On the current stream (``stream`` left out) a product is one call into the library's Python module, with the operands it
quantizes in a buffer of its own: codes and scales are those of the calls one by one, and so are the products, except that
``fprop`` of few rows (``few_rows_in_one_launch`` in csrc/gemm_shapes.hpp) finds scale, codes and product in one launch whose waves share K
another way.  There the fp32 sums are added in another order than ``nvfp4_46_gemm`` adds them, and an output can be the
neighbouring BF16 value of the one that the same call with ``stream=`` returns.  On any other stream, and for operands that are
not plain contiguous tensors, a product is those calls one by one.

Every function takes an optional ``workspace`` (``binding.new_workspace()``).  With it, and on the default stream also without,
a tensor scale is one launch; on another stream without a workspace it is three.  ``wgrad`` on the current stream finds the
scales of its two operands in one launch and their codes in a second where such scratch words are at hand and the operands
are not too large for it (``nvfp4_46_wgrad_operands`` in csrc/nvfp4_46.hip).  One workspace serves all calls issued on one stream.
"""
from __future__ import annotations

import torch

from . import binding as B


def quantize_weight(w: torch.Tensor, select: int = B.SEL_46_MSE, block2d: bool = True,
                    stream=None, workspace: torch.Tensor | None = None) -> dict:
    """W [N][K] (FP32 master copy or BF16) -> both packings and the tensor scale."""
    q = B.nvfp4_46_scale_quantize(w, workspace, layout=B.BOTH, select=select, want_choice=False,
                                  block2d=int(block2d), stream=stream)
    q.update(block2d=bool(block2d), shape=tuple(w.shape))
    return q


def _rowwise(t, stream, workspace, **kw):
    q = B.nvfp4_46_scale_quantize(t, workspace, want_choice=False, stream=stream, **kw)
    return q["codes_row"], q["scales_row"], q["alpha"]


def _columnwise(t, stream, workspace, rht_seed, **kw):
    q = B.nvfp4_46_scale_quantize(t, workspace, layout=B.COLWISE, rht=1, rht_seed=rht_seed,
                                  want_choice=False, stream=stream, **kw)
    return q["codes_col"], q["scales_col"], q["alpha"]


def fprop(x: torch.Tensor, qw: dict, select: int = B.SEL_46_MSE, stream=None,
          workspace: torch.Tensor | None = None) -> torch.Tensor:
    """y [T][N] BF16 = x W^T."""
    flags = B.GEMM_B_TILE_SCALES if qw["block2d"] else 0
    if stream is None:
        y = B.product_of_rows(x, qw["codes_row"], qw["scales_row"], qw["alpha"], flags, B.RTN, select, 0, workspace)
        if y is not None:
            return y
    cx, sx, ax = _rowwise(x, stream, workspace, select=select)
    return B.nvfp4_46_gemm(cx, sx, ax, qw["codes_row"], qw["scales_row"], qw["alpha"],
                           out_dtype=B.OUT_BF16, flags=flags, stream=stream)


def dgrad(dy: torch.Tensor, qw: dict, sr_seed: int, select: int = B.SEL_46_MSE,
          stream=None, workspace: torch.Tensor | None = None) -> torch.Tensor:
    """dx [T][K] BF16 = dy W, the gradient rounded stochastically."""
    flags = B.GEMM_B_TILE_SCALES if qw["block2d"] else 0
    if stream is None:
        dx = B.product_of_rows(dy, qw["codes_col"], qw["scales_col"], qw["alpha"], flags, B.SR, select, sr_seed, workspace)
        if dx is not None:
            return dx
    cg, sg, ag = _rowwise(dy, stream, workspace, select=select, rounding=B.SR, sr_seed=sr_seed)
    return B.nvfp4_46_gemm(cg, sg, ag, qw["codes_col"], qw["scales_col"], qw["alpha"],
                           out_dtype=B.OUT_BF16, flags=flags, stream=stream)


def wgrad(dy: torch.Tensor, x: torch.Tensor, sr_seed: int, rht_seed: int,
          select: int = B.SEL_46_MSE, stream=None,
          workspace: torch.Tensor | None = None) -> torch.Tensor:
    """dW [N][K] FP32 = dy^T x, both operands Hadamard-transformed along the token axis."""
    if stream is None:
        dw = B.product_of_columns(dy, x, sr_seed, rht_seed, select, workspace)
        if dw is not None:
            return dw
    cg, sg, ag = _columnwise(dy, stream, workspace, rht_seed, select=select, rounding=B.SR,
                             sr_seed=sr_seed)
    cx, sx, ax = _columnwise(x, stream, workspace, rht_seed, select=select)
    return B.nvfp4_46_gemm(cg, sg, ag, cx, sx, ax, out_dtype=B.OUT_F32, stream=stream)
