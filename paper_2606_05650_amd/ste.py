"""The codec as a differentiable layer (straight-through quantizer).

SteCoder.apply(attr, pos, params) runs the HIP encoder through gsc_ste_forward and returns, for
the Nv occupied voxels in Morton order, the dequantized coefficients yhat, the decoded
attributes ahat = T^T yhat and the voxel means aref (not differentiable). Its backward runs
gsc_ste_backward: the quantizer passes gradients unchanged, the transform's adjoint (the
inverse RAHT) maps them back to voxels, and each Gaussian receives its voxel's gradient divided
by the voxel's member count. Nv is only known once the encoder has run, so this form waits for
the device to cut the outputs to Nv rows.

SteCoderPadded.apply(attr, pos, params) is the same layer without that wait, for training loops
that must not stall on the device: it returns n rows (rows past Nv zero) and Nv as a one-element
device tensor. Nothing in its forward or backward synchronizes the host. A device-detected error
(corrupt input, capacity) leaves Nv = 0 and every row zero, which makes rd_loss's distortion NaN.

rd_loss is the rate-distortion objective of the differentiable workload: the mean squared error
of the decoded attributes against the voxel means plus lambda times the rate proxy
sum log2(1 + |yhat| / step). On plain contiguous float32 device rows it runs fused: one pass
forward and one backward for each term (_RdDist, _RdRate); every other call is the same formula in torch operators.
"""
from __future__ import annotations

import math

import torch

from . import gsc


def _backward(ctx, g_yhat, g_ahat):
    fwd = ctx.fwd
    C = fwd.encoded.C
    dev = fwd.yhat.device
    z = None
    if g_yhat is None or g_ahat is None:
        z = torch.zeros((max(fwd.n, 1), C), dtype=torch.float32, device=dev)
    gy = z if g_yhat is None else g_yhat.float().contiguous()
    ga = z if g_ahat is None else g_ahat.float().contiguous()
    # the kernels read rows < Nv of the gradients (Nv from the workspace, on the device)
    grad, _info = gsc.ste_backward(fwd, gy, ga)
    return grad[:fwd.n]


class SteCoder(torch.autograd.Function):
    @staticmethod
    def forward(ctx, attr, pos, params):
        if not attr.is_cuda:
            raise ValueError("SteCoder runs on the GPU only")
        fwd = gsc.ste_forward(pos.contiguous(), attr.detach().contiguous(), params)
        fwd.encoded.check()                 # synchronizes: Nv sizes the outputs
        nv = fwd.encoded.n_vox()
        ctx.fwd = fwd
        aref = fwd.aref[:nv]
        ctx.mark_non_differentiable(aref)
        return fwd.yhat[:nv], fwd.ahat[:nv], aref

    @staticmethod
    def backward(ctx, g_yhat, g_ahat, _g_aref):
        return _backward(ctx, g_yhat, g_ahat), None, None


class SteCoderPadded(torch.autograd.Function):
    @staticmethod
    def forward(ctx, attr, pos, params):
        if not attr.is_cuda:
            raise ValueError("SteCoderPadded runs on the GPU only")
        n = int(pos.shape[0])
        # the kernels write rows below Nv; the rest is cleared once Nv is known on the device
        fwd = gsc.ste_forward(pos.contiguous(), attr.detach().contiguous(), params)
        nv = gsc.ste_pad(fwd)
        z = (fwd.yhat, fwd.ahat, fwd.aref)
        if n == 0:
            for t in z:  # (one row is allocated)
                t.zero_()
        ctx.fwd = fwd
        out = [t[:n] for t in z]
        ctx.mark_non_differentiable(out[2], nv)
        return out[0], out[1], out[2], nv

    @staticmethod
    def backward(ctx, g_yhat, g_ahat, _g_aref, _g_nv):
        return _backward(ctx, g_yhat, g_ahat), None, None


class _RdDist(torch.autograd.Function):
    """The distortion of a fused forward (gsc.rd_loss_forward's results) by ahat. The difference ahat - aref
    is an output of its own, so that neither ahat nor aref has to stay unchanged until the backward,
    and so that gradients of the gradient flow through it."""

    @staticmethod
    def forward(ctx, ahat, results):
        ctx.set_materialize_grads(False)
        _, dist, _, ctx.count, diff = results
        ctx.save_for_backward(diff)
        return dist, diff

    @staticmethod
    def backward(ctx, g_dist, g_diff):
        (diff,) = ctx.saved_tensors  # (as a saved-tensor hook hands it back)
        if g_dist is None:
            return g_diff, None
        if not torch.is_grad_enabled() and g_diff is None and _readable(diff, diff.device) and _readable(g_dist, diff.device):
            return gsc.rd_loss_backward(None, diff, None, 0.0, ctx.count, None, g_dist, None)[1], None
        # differentiable (create_graph), a gradient of the difference, or tensors that are not plain
        # memory (batched gradients): torch operators
        ga = g_dist * 2.0 * diff / (ctx.count * diff.shape[1])
        return ga if g_diff is None else ga + g_diff, None


class _RdRate(torch.autograd.Function):
    """The rate of a fused forward by yhat."""

    @staticmethod
    def forward(ctx, yhat, steps, lam, results):
        ctx.set_materialize_grads(False)
        ctx.lam = lam
        ctx.save_for_backward(yhat, steps)
        return results[2]

    @staticmethod
    def backward(ctx, g_rate):
        yhat, steps = ctx.saved_tensors
        if g_rate is None:
            return None, None, None, None
        if not torch.is_grad_enabled() and all(_readable(t, yhat.device) for t in (yhat, steps, g_rate)):
            return gsc.rd_loss_backward(yhat, None, steps, ctx.lam, None, None, None, g_rate)[0], None, None, None
        return g_rate * (ctx.lam / math.log(2.0)) * yhat.sgn() / (steps + yhat.abs()), None, None, None


def _readable(t, device, dtype=torch.float32):
    """Whether a kernel may read t's memory as it stands: an ordinary dense tensor of the type, and not
    a transform's wrapper (which has no memory of its own) or a view that negates when it is read."""
    if type(t) not in (torch.Tensor, torch.nn.Parameter) or t.dtype != dtype or t.device != device:
        return False
    if t.layout != torch.strided or not t.is_contiguous() or t.is_neg():
        return False
    try:
        return t.data_ptr() != 0
    except RuntimeError:
        return False


def _watched():
    """Whether a compiler, a trace, a transform, forward mode or a mode is active that has to see the
    operators. torch has no public name for most of these questions: where one cannot be asked, the
    answer is yes."""
    try:
        return (torch.compiler.is_compiling() or torch.jit.is_tracing() or
                torch._C._are_functorch_transforms_active() or torch.autograd.forward_ad._current_level >= 0 or
                torch._C._len_torch_dispatch_stack() > 0 or torch._C._len_torch_function_stack() > 0)
    except AttributeError:
        return True


def _plain_rows(yhat, ahat, aref, steps, lam, nv):
    """Whether rd_loss may run fused: ordinary float32 rows on the current device, gradients
    wanted of yhat and ahat only, and no mode or transform active that has to see the operators."""
    ts = (yhat, ahat, aref, steps) + (() if nv is None else (nv,))
    if not all(isinstance(t, torch.Tensor) for t in ts) or type(lam) not in (int, float):
        return False
    if not yhat.is_cuda or yhat.device.index != torch.cuda.current_device():
        return False
    if yhat.dim() != 2 or not 1 <= yhat.shape[0] <= gsc.MAX_ROWS or not 1 <= yhat.shape[1] <= gsc.MAX_CHANNELS:
        return False
    if not all(_readable(t, yhat.device) for t in ts[:4]) or any(t.shape != yhat.shape for t in ts[1:3]):
        return False
    if steps.shape != yhat.shape[1:] or aref.requires_grad or steps.requires_grad:
        return False
    if nv is not None and (nv.numel() != 1 or not _readable(nv, yhat.device, torch.int64)):
        return False
    return not _watched()


def rd_loss(yhat, ahat, aref, steps, lam, nv=None):
    """(loss, distortion, rate): mean((ahat - aref)^2) + lam * sum(log2(1 + |yhat| / steps)).

    With nv (SteCoderPadded's device count) the rows are the padded ones: the mean is taken over
    the nv voxel rows (the zero rows past them add nothing to either term), with no host wait."""
    if _plain_rows(yhat, ahat, aref, steps, lam, nv):
        of_yhat, of_ahat = (torch.is_grad_enabled() and t.requires_grad for t in (yhat, ahat))
        results = gsc.rd_loss_forward(yhat, ahat, aref, steps, lam, nv=nv, want_diff=of_ahat)
        loss, dist, rate = results[:3]
        # (the terms' graphs are their own: each may be differentiated alone, once)
        if of_ahat:
            dist, _ = _RdDist.apply(ahat, results)
        if of_yhat:
            rate = _RdRate.apply(yhat, steps, lam, results)
        return dist + rate if of_yhat or of_ahat else loss, dist, rate
    sq = (ahat - aref) ** 2
    r = torch.log2(1.0 + yhat.abs() / steps)
    if nv is None:
        dist = sq.mean()
    else:
        dist = sq.sum() / (nv.to(sq.dtype) * sq.shape[1]).reshape(())
    rate = lam * r.sum()
    return dist + rate, dist, rate
