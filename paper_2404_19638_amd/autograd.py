"""Hand-written backward passes of the local hot path (torch.autograd).

Every forward and backward step is a call into libspc3d; PyTorch only holds
the tensors and records the graph.  The gradients follow from the two
definitions (Eq. (1) and Eq. (2) of the paper) by the chain rule, and each is
itself one of the library's kernels:

  SDDMM   c_p = s_p <a_i, b_j>      (i = row, j = column of slot p)
          dA  = SpMM(S o dC, B)            dB  = SpMM^T(S o dC, A)
          ds  = SDDMM(dC, A, B)            (sampling values dC_p)
  SpMM    y_i = sum_p s_p b_j
          dB  = SpMM^T(S, dY)              ds  = SDDMM(pattern, dY, B)
  softmax alpha = rowsoftmax(e)            de  = alpha o (dalpha - rowsum(alpha o dalpha))
  gather  packed = src[gmap]               dsrc = scatter-add(dpacked)
  scatter dst += packed[...]               dpacked = gather(ddst)

Gradients with respect to A and B of the transposed SpMM need the plan's
column-major view (SPC3D_BUILD_CSC).

Dense operands may be bfloat16 (the library accumulates in FP32): outputs
are FP32, the upstream gradient of a product with bfloat16 operands is
rounded to bfloat16 before it enters the backward kernels (half the bytes
per gathered row), and each returned gradient has its input's type.
"""
from __future__ import annotations

import torch

from . import spc3d as spc


def _needs(ctx, i):
    return ctx.needs_input_grad[i]


# Stored entries up to which the transposed SpMM reads its values through the
# slot map.  us through the map / permuted first (permute + SpMM; MI355X, R-MAT
# of degree 32, FP32): 1.8M entries kz = 32 31.7 / 37.8, kz = 64 42.6 / 48.6; 7.6M
# 129 / 144, 205 / 206; 31.4M 755 / 669, 1530 / 989 (the 126 MB of values miss L2,
# once per slice).  At 53,000 entries 9.2 / 13.7: a launch less.
DIRECT_MAX_NNZ = 1 << 22


def _spmm_t(plan, vals, X):
    """Transposed SpMM (sum over each column's entries).  On large blocks the
    values are first permuted to column-major order so the kernel reads them as
    one stream rather than one random load per entry through the slot map (the
    same results, bit for bit)."""
    if vals is None or plan.nnz <= DIRECT_MAX_NNZ:
        return spc.spmm(plan, vals, X, transpose=1)
    vt = spc.permute_values(plan, spc.SLOT_TO_COLUMN, vals)
    return spc.spmm(plan, vt, X, transpose=2)


def _as(grad, like):
    """A gradient (FP32 from the library) in the type of its input: with
    bfloat16 operands the products still accumulate in FP32 and only the
    returned gradient is rounded."""
    return grad if grad.dtype == like.dtype else grad.to(like.dtype)


class SDDMMFn(torch.autograd.Function):
    """out = SDDMM(plan, vals, A, B); vals None means pattern-only (s == 1)."""

    @staticmethod
    def forward(ctx, plan, vals, A, B):
        ctx.plan = plan
        # the kernels take packed operands: a sliced input (e.g. a column block
        # of a wider tensor) is copied once and the copy serves both passes
        vals = None if vals is None else vals.contiguous()
        A, B = A.contiguous(), B.contiguous()
        ctx.save_for_backward(vals if vals is not None else torch.empty(0), A, B)
        ctx.has_vals = vals is not None
        return spc.sddmm(plan, vals, A, B)

    @staticmethod
    def backward(ctx, dout):
        plan = ctx.plan
        vals, A, B = ctx.saved_tensors
        dout = dout.contiguous()
        w = spc.mul_values(plan, dout, vals) if ctx.has_vals else dout
        dvals = dA = dB = None
        if ctx.has_vals and _needs(ctx, 1):
            dvals = spc.sddmm(plan, dout, A, B)
        if _needs(ctx, 2):
            dA = _as(spc.spmm(plan, w, B, transpose=0), A)
        if _needs(ctx, 3):
            dB = _as(_spmm_t(plan, w, A), B)
        return None, dvals, dA, dB


class SpMMFn(torch.autograd.Function):
    """Y = SpMM(plan, vals, X) over rows (transpose 0) or columns (transpose 1)."""

    @staticmethod
    def forward(ctx, plan, vals, X, transpose=0):
        ctx.plan = plan
        ctx.transpose = transpose
        ctx.has_vals = vals is not None
        vals = None if vals is None else vals.contiguous()
        X = X.contiguous()
        ctx.save_for_backward(vals if vals is not None else torch.empty(0), X)
        return spc.spmm(plan, vals, X, transpose=transpose)

    @staticmethod
    def backward(ctx, dY):
        plan = ctx.plan
        vals, X = ctx.saved_tensors
        dY = dY.contiguous()
        dvals = dX = None
        dYx = dY.to(X.dtype)   # the upstream gradient in X's type (bfloat16 rows gather half the bytes)
        if ctx.has_vals and _needs(ctx, 1):
            # d y_i / d s_p = x_j: one dot per slot
            if ctx.transpose == 0:
                dvals = spc.sddmm(plan, None, dYx, X)
            else:
                dvals = spc.sddmm(plan, None, X, dYx)
        if _needs(ctx, 2):
            v = vals if ctx.has_vals else None
            if ctx.transpose == 0:
                dX = _as(_spmm_t(plan, v, dYx), X)
            else:
                dX = _as(spc.spmm(plan, v, dYx, transpose=0), X)
        return None, dvals, dX, None


class RowSoftmaxFn(torch.autograd.Function):
    @staticmethod
    def forward(ctx, plan, e):
        alpha = spc.row_softmax(plan, e.contiguous())
        ctx.plan = plan
        ctx.save_for_backward(alpha)
        return alpha

    @staticmethod
    def backward(ctx, dalpha):
        (alpha,) = ctx.saved_tensors
        return None, spc.row_softmax_bwd(ctx.plan, alpha, dalpha.contiguous())


class GatherFn(torch.autograd.Function):
    """packed = rows gmap[l] - lo of src, columns [k0, k0+kz) (FP32)."""

    @staticmethod
    def forward(ctx, plan, axis, src, k0, kz):
        ctx.plan, ctx.axis, ctx.k0, ctx.shape = plan, axis, k0, src.shape
        return spc.gather(plan, axis, src, k0, kz)

    @staticmethod
    def backward(ctx, dpacked):
        dsrc = torch.zeros(ctx.shape, dtype=torch.float32, device=dpacked.device)
        spc.scatter_reduce(ctx.plan, ctx.axis, dpacked.contiguous(), dsrc, ctx.k0)
        return None, None, dsrc, None, None


class ScatterReduceFn(torch.autograd.Function):
    """Returns dst + (packed rows added at gmap rows, columns k0..k0+kz)."""

    @staticmethod
    def forward(ctx, plan, axis, packed, dst, k0):
        ctx.plan, ctx.axis, ctx.k0, ctx.kz = plan, axis, k0, packed.shape[1]
        out = dst.clone()
        spc.scatter_reduce(plan, axis, packed.contiguous(), out, k0)
        return out

    @staticmethod
    def backward(ctx, dout):
        dout = dout.contiguous()
        dpacked = spc.gather(ctx.plan, ctx.axis, dout, ctx.k0, ctx.kz)
        return None, None, dpacked, dout, None


def _attention_bwd(needs, plan, alpha, dout, Q, Kf, V):
    """(dQ, dKf, dV) of out = alpha . V, alpha = rowsoftmax(SDDMM(Q, Kf)); None
    where not needed.  On blocks beyond DIRECT_MAX_NNZ whose two transposed
    products both follow, one pass takes alpha and de to column order."""
    dout = dout.to(V.dtype)   # the upstream gradient in the operands' type
    dQ = dK = dV = de = at = det = None
    if needs[0] or needs[1]:
        dalpha = spc.sddmm(plan, None, dout, V)
        if needs[1] and needs[2] and plan.nnz > DIRECT_MAX_NNZ:
            de, at, det = spc.row_softmax_bwd_columns(plan, alpha, dalpha, out=dalpha)
        else:
            de = spc.row_softmax_bwd(plan, alpha, dalpha, out=dalpha)
    if needs[0]:
        dQ = _as(spc.spmm(plan, de, Kf, transpose=0), Q)
    if needs[1]:
        dK = _as(_spmm_t(plan, de, Q) if det is None
                 else spc.spmm(plan, det, Q, transpose=2), Kf)
    if needs[2]:
        dV = _as(_spmm_t(plan, alpha, dout) if at is None
                 else spc.spmm(plan, at, dout, transpose=2), V)
    return dQ, dK, dV


class AttentionFn(torch.autograd.Function):
    """out = rowsoftmax(SDDMM(pattern, Q, Kf)) . V in the three kernels, with
    alpha kept for the backward."""

    @staticmethod
    def forward(ctx, plan, Q, Kf, V):
        Q, Kf, V = Q.contiguous(), Kf.contiguous(), V.contiguous()
        alpha = spc.row_softmax(plan, spc.sddmm(plan, None, Q, Kf))
        ctx.plan = plan
        ctx.save_for_backward(Q, Kf, V, alpha)
        return spc.spmm(plan, alpha, V)

    @staticmethod
    def backward(ctx, dout):
        Q, Kf, V, alpha = ctx.saved_tensors
        return None, *_attention_bwd(ctx.needs_input_grad[1:], ctx.plan, alpha,
                                     dout.contiguous(), Q, Kf, V)


class FusedAttentionFn(torch.autograd.Function):
    """out = rowsoftmax(SDDMM(pattern, Q, Kf)) . V in one fused pass
    (spc3d_attention_fwd).  The backward recomputes the scores with one SDDMM,
    rebuilds alpha from the stored row (max, sum) pairs, and then runs the
    chain of the unfused layer: dalpha = SDDMM(dout, V), de = softmax
    backward, dQ = SpMM(de, Kf), dKf = SpMM^T(de, Q), dV = SpMM^T(alpha, dout)."""

    @staticmethod
    def forward(ctx, plan, Q, Kf, V):
        Q, Kf, V = Q.contiguous(), Kf.contiguous(), V.contiguous()
        out, stats = spc.attention_fwd(plan, Q, Kf, V)
        ctx.plan = plan
        ctx.save_for_backward(Q, Kf, V, stats)
        return out

    @staticmethod
    def backward(ctx, dout):
        plan = ctx.plan
        Q, Kf, V, stats = ctx.saved_tensors
        e = spc.sddmm(plan, None, Q, Kf)
        alpha = spc.row_softmax_apply(plan, e, stats, out=e)
        return None, *_attention_bwd(ctx.needs_input_grad[1:], plan, alpha, dout.contiguous(),
                                     Q, Kf, V)


def sddmm(plan, vals, A, B):
    return SDDMMFn.apply(plan, vals, A, B)


def spmm(plan, vals, X, transpose=0):
    return SpMMFn.apply(plan, vals, X, transpose)


def row_softmax(plan, e):
    return RowSoftmaxFn.apply(plan, e)


def gather(plan, axis, src, k0, kz):
    return GatherFn.apply(plan, axis, src, k0, kz)


def scatter_reduce(plan, axis, packed, dst, k0):
    return ScatterReduceFn.apply(plan, axis, packed, dst, k0)


def _need_fused(Q, Kf, V):
    dt = spc.BF16 if Q.dtype == torch.bfloat16 else spc.F32
    if not spc.attention_supported(Q.shape[1], dt):
        raise ValueError(f"the fused attention pass does not cover K={Q.shape[1]}")
    if not all(t.data_ptr() % 16 == 0 for t in (Q, Kf, V)):
        raise ValueError("the fused attention pass needs 16-byte aligned Q, Kf and V")


# Largest block (stored entries) on which the automatic choice takes the
# one-pass forward, by the bytes of a row of Kf: its two rows a slot are live
# together, so wide rows outgrow the caches earlier than the three kernels, which
# also take wide rows of skewed columns in slices.  us three kernels / one pass
# (MI355X, R-MAT): 128-byte rows gain at every size (FP32 K = 32, 1.8M entries
# 64.9 / 45.1, 31.4M 782 / 773; bfloat16 K = 64 871 / 811).  256 bytes: FP32 2.8M
# 128 / 120, 3.0M 144 / 147, 7.6M 314 / 336; bfloat16 K = 128 7.6M 369 / 357, 15.5M
# 763 / 825.  512 bytes: FP32 K = 128 883,000 82.4 / 77.3, 955,000 92.6 / 97.8, 1.8M
# 147 / 162; bfloat16 K = 256 955,000 111 / 108, 7.6M 663 / 871.  On uniform and
# banded blocks the two differ less: 64- and 128-byte rows 0.91 to 1.99 times as
# fast in one pass from 300,000 to 16M entries (FP32 K = 32: uniform 8M, 20 a row,
# 364 / 344, banded 5M 148 / 133; the losses: banded 2.6M, half-width 20,000, 98 /
# 108, K = 16 banded 7.8M 269 / 295, uniform 4M, 33 a row, 117 / 124, R-MAT 2^20,
# 16M, 378 / 405), 256 bytes on either side of the line 0.97 to 1.10 (FP32 uniform
# 2M 173 / 161, banded 2M 103 / 98, uniform 2.6M 229 / 216, 16M 1282 / 1269) but
# for banded blocks past it (5M 308 / 261).
AUTO_FUSED_F32_MAX_NNZ = 1 << 21
_AUTO_FUSED_MAX_NNZ = {(spc.F32, 256): AUTO_FUSED_F32_MAX_NNZ, (spc.F32, 512): 900_000,
                       (spc.BF16, 256): 1 << 23, (spc.BF16, 512): 1 << 20}


def _auto_fused(plan, Q, Kf, V):
    """The forward gnn_attention takes when the caller leaves it open: the
    one-pass kernel for inference (no gradient is recorded) where it measured
    faster, the three kernels otherwise (the fused backward recomputes the
    scores, and the fused forward loses with wide rows on large blocks)."""
    if torch.is_grad_enabled() and any(t.requires_grad for t in (Q, Kf, V)):
        return False
    if not (Q.dtype == Kf.dtype == V.dtype) or Q.dtype not in (torch.float32, torch.bfloat16):
        return False
    dt = spc.BF16 if Q.dtype == torch.bfloat16 else spc.F32
    if not spc.attention_supported(Q.shape[1], dt):
        return False
    if not all(t.is_contiguous() and t.data_ptr() % 16 == 0 for t in (Q, Kf, V)):
        return False
    limit = _AUTO_FUSED_MAX_NNZ.get((dt, Q.shape[1] * Q.element_size()))
    return limit is None or plan.nnz <= limit


def gnn_attention(plan, Q, Kf, V, fused: bool | None = None):
    """Masked attention over the block's pattern: SDDMM edge scores (s == 1),
    row softmax over each row's stored entries, SpMM aggregation of V.

    Q is [R, K] (local rows), Kf and V are [C, K] (local columns); returns [R, K].
    fused=True runs the forward as one pass (spc3d_attention_fwd; K must be
    covered by it, see spc.attention_supported) and recomputes the scores in
    the backward; fused=False runs the three separate kernels.  Left as None,
    the one-pass forward is taken for inference (no gradient recorded) where it
    measured faster: rows of up to 128 bytes on every block, wider ones up to a
    number of entries (see _AUTO_FUSED_MAX_NNZ), and the three kernels otherwise.

    Memory: the backward of a block beyond DIRECT_MAX_NNZ entries whose Kf and V
    both need gradients holds four FP32 values an entry (alpha and the score
    gradients in column order, and the pairs they are taken from) besides alpha
    and the score gradients themselves; otherwise one.
    """
    if fused is None:
        fused = _auto_fused(plan, Q, Kf, V)
    if fused:
        _need_fused(Q, Kf, V)
        return FusedAttentionFn.apply(plan, Q, Kf, V)
    return AttentionFn.apply(plan, Q, Kf, V)
