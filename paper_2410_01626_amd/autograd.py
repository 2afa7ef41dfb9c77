"""torch.autograd wrapper of the solver: forward = fmm_eval, backward = one of
the library's adjoint calls, which rebuild the octree and every expansion
from the saved inputs instead of storing them.

E, F and phi are differentiable; dV/dlambda is returned as a
non-differentiable output.  For an upstream weight w on E alone,
fmm_eval_adjoint returns
    dE/dx = -w F,  dE/dqA = w (1 - lambda_s) phi,  dE/dqB = w lambda_s phi,
    dE/dlambda = w dV/dlambda
(sites -1: dE/dqA = w phi, dE/dqB = 0); with weights on phi or F (whatever their
values: none is looked at, backward never waits for the device),
fmm_eval_adjoint_full returns the gradient of w E + gphi . phi + gF . F in one
tree pass (charges and, as second sources, charges gphi with dipoles -q gF).
"""
from __future__ import annotations

import torch


def _fork(plan, device):
    """A plan on another stream than autograd's: its kernels run after the work
    queued here so far (their inputs, the memory of their outputs) and, by
    _join, the work queued here afterwards runs after them (readers of the
    outputs, whoever is given the memory of a tensor freed here next).  Waits
    between the streams, none on the host; under capture the plan's stream joins
    and leaves.  Returns None for a plan on this stream (the usual case, told by
    the bare handle: stream objects cost 20 us of a 200 us gradient)."""
    if torch._C._cuda_getCurrentRawStream(plan.device.index) == plan.stream.cuda_stream:
        return None
    here = torch.cuda.current_stream(device)
    there = torch.cuda.ExternalStream(plan.stream.cuda_stream, device=device)
    there.wait_stream(here)
    return here, there


def _join(streams):
    if streams is not None:
        streams[0].wait_stream(streams[1])


class FmmCoulomb(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, qA, qB, lam, plan, site, box):
        streams = _fork(plan, x.device)
        try:
            out = plan.eval(x, qA, qB, site, lam, box=box)
        finally:
            _join(streams)
        ctx.save_for_backward(x, qA, qB, lam, site)
        ctx.plan = plan
        ctx.box = box
        ctx.mark_non_differentiable(out["dVdl"])
        # outputs the loss does not use arrive as None in backward, not as zeros
        # that only a wait for the device could tell from weights
        ctx.set_materialize_grads(False)
        return out["E"], out["F"], out["phi"], out["dVdl"]

    @staticmethod
    def backward(ctx, gE, gF, gphi, gdVdl):
        if gdVdl is not None and bool(torch.any(gdVdl != 0)):
            raise NotImplementedError("dV/dlambda is not differentiable; got a gradient on it")
        x, qA, qB, lam, site = ctx.saved_tensors
        w = None if gE is None else gE.to(torch.float64).reshape(1).contiguous()
        gphi = None if gphi is None else gphi.to(x.dtype).contiguous()
        gF = None if gF is None else gF.to(x.dtype).contiguous()
        if w is None and gphi is None and gF is None:
            w = torch.zeros(1, dtype=torch.float64, device=x.device)
        streams = _fork(ctx.plan, x.device)
        try:
            if gphi is not None or gF is not None:
                adj = ctx.plan.eval_adjoint_full(x, qA, qB, site, lam, gE=w, gphi=gphi, gF=gF, box=ctx.box)
            else:
                adj = ctx.plan.eval_adjoint(x, qA, qB, site, lam, w, box=ctx.box)
        finally:
            _join(streams)
        return (adj["grad_x"] if ctx.needs_input_grad[0] else None,
                adj["grad_qA"] if ctx.needs_input_grad[1] else None,
                adj["grad_qB"] if ctx.needs_input_grad[2] else None,
                adj["grad_lambda"] if ctx.needs_input_grad[3] else None,
                None, None, None)


def fmm_coulomb(plan, x, qA, qB, site, lam, box=None):
    """Differentiable energy, forces and potential (and non-differentiable
    dV/dlambda)."""
    E, F, phi, dVdl = FmmCoulomb.apply(x, qA, qB, lam, plan, site, box)
    return E, F, phi, dVdl
