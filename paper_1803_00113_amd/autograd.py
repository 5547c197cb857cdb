"""torch.autograd.Function over the library's ELBO (the adjoint kernel of the pixel path).

elbo(plan, theta), where a gradient can be wanted (gradient mode on, theta requiring it):
forward:  cel_elbo_grad -- one evaluation gives the value and the gradient, which is kept with
          the graph
backward: the kept gradient scaled by the incoming one
A value and its gradient by cel_elbo_eval in the forward and cel_elbo_grad in the backward are
two evaluations with the same tables, moment maps and pixel values: 137 us for a star and a
galaxy on 32 x 32 cutouts against 101 us in one.  The objective is the same bit for bit.

A value alone costs less than a value with its gradient (330 against 432 us for 1000 sources).
Without a backward (line searches, logging, validation) call elbo under torch.no_grad() or
with theta.detach(); where a backward may or may not follow, ElboFunction.apply(theta, plan)
evaluates the value and leaves the gradient to the backward.
"""
import torch

from . import api


class ElboFunction(torch.autograd.Function):
    """apply(theta, plan, with_grad=False): with_grad forms the gradient in the forward."""

    @staticmethod
    def forward(ctx, theta, plan, with_grad=False):
        if with_grad:
            tot, _, g = api.elbo_grad(plan, theta.detach())
            ctx.save_for_backward(theta, g)   # (theta: its version is checked in the backward)
        else:
            tot, _ = api.elbo_eval(plan, theta.detach())
            ctx.save_for_backward(theta)
            ctx.plan = plan
        return tot.reshape(())

    @staticmethod
    def backward(ctx, grad_out):
        theta, *kept = ctx.saved_tensors
        g = kept[0] if kept else api.elbo_grad(ctx.plan, theta.detach())[2]
        return (grad_out * g.to(theta.dtype),) + (None,) * (len(ctx.needs_input_grad) - 1)


def elbo(plan, theta):
    """Global ELBO of `plan` at theta [S,32] (float64 cuda) as a differentiable scalar."""
    return ElboFunction.apply(theta, plan, torch.is_grad_enabled() and theta.requires_grad)
