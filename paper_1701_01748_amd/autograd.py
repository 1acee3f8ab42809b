"""Differentiable measurement and sparsity operators, and unrolled PPD.

The forward and backward passes of the linear operators are the library's
HIP kernels: the adjoint of `Phi` (Sec. 2) is the gridding path
`Re Phi^H`, and the SARA analysis and synthesis (Sec. 5.1) are each other's
adjoint (Psi Psi^H = I, real).  Torch's convention for a real loss L of a
complex tensor y is grad = dL/dRe(y) + i dL/dIm(y); with it

    y = Phi x (x real)   ->  grad_x = Re(Phi^H grad_y)
    x = Re(Phi^H y)      ->  grad_y = Phi grad_x

`unrolled_ppd` composes K iterations of Algorithm 3 from these operators and
the library's three updates (data dual, sparsity dual, primal), whose
backward passes are the library's VJP kernels: the l2-ball projection's
Jacobian per block, the clip mask and the positivity mask (the proximity
operators are piecewise smooth).  Each iteration can be checkpointed, so
memory stays at one iteration's activations.

A whole iteration, and the data fidelity of all channels, are one autograd
node each: composed of the pieces' nodes and torch operations the calls are
bound by the host, whose speed differs from process to process.  Medians of
separate runs: an iteration at 256^2, 65536 points, forward and backward 412 to
533 us, as one node 249 to 427; the fidelity of four channels of 250000 points
at 512^2 with its gradient 741 to 855 us, as one node 211 to 269.
"""
from __future__ import annotations

from typing import Optional, Sequence

import torch
import torch.autograd.forward_ad as fwAD
import torch.utils.checkpoint

from . import ppd as P


class PhiFn(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, plan):
        ctx.plan = plan
        return P.ppd_phi(plan, x.detach().contiguous().to(torch.float32))

    @staticmethod
    def backward(ctx, g):
        return P.ppd_phit(ctx.plan, g.contiguous().to(torch.complex64)), None


class PhitFn(torch.autograd.Function):
    @staticmethod
    def forward(ctx, y, plan):
        ctx.plan = plan
        return P.ppd_phit(plan, y.detach().contiguous().to(torch.complex64))

    @staticmethod
    def backward(ctx, g):
        return P.ppd_phi(ctx.plan, g.contiguous().to(torch.float32)), None


class SaraAnalysisFn(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, plan):
        ctx.plan = plan
        return P.ppd_sara(plan, P.SARA_ANALYSIS, x.detach().contiguous().to(torch.float32))

    @staticmethod
    def backward(ctx, g):
        return P.ppd_sara(ctx.plan, P.SARA_SYNTHESIS, g.contiguous().to(torch.float32)), None


class SaraSynthesisFn(torch.autograd.Function):
    @staticmethod
    def forward(ctx, u, plan):
        ctx.plan = plan
        return P.ppd_sara(plan, P.SARA_SYNTHESIS, u.detach().contiguous().to(torch.float32))

    @staticmethod
    def backward(ctx, g):
        return P.ppd_sara(ctx.plan, P.SARA_ANALYSIS, g.contiguous().to(torch.float32)), None


def phi(plan, x):
    """y = Theta G F Z x, differentiable (plan order)."""
    return PhiFn.apply(x, plan)


def phit(plan, y):
    """x = Re Phi^H y, differentiable."""
    return PhitFn.apply(y, plan)


def sara_analysis(plan, x):
    return SaraAnalysisFn.apply(x, plan)


def sara_synthesis(plan, u):
    return SaraSynthesisFn.apply(u, plan)


class FidelityFn(torch.autograd.Function):
    """sum_c ||Phi_c x - y_c||^2 for constant data y_c, one node for all
    channels; backward: 2 sum_c Re Phi_c^H r_c."""

    @staticmethod
    def forward(ctx, x, plans, ys):
        xd = x.detach().contiguous().to(torch.float32)
        acc = torch.empty(1, dtype=torch.float64, device=xd.device)
        loss = torch.empty((), dtype=torch.float32, device=xd.device)
        rs = [P.ppd_fidelity(p, xd, y.detach(), acc, loss, k > 0) for k, (p, y) in enumerate(zip(plans, ys))]
        ctx.plans = plans
        ctx.save_for_backward(*rs)
        return loss

    @staticmethod
    def backward(ctx, g):
        rs = [_dense(r, torch.complex64) for r in ctx.saved_tensors]   # as saved-tensor hooks hand them back
        img = P.ppd_phit(ctx.plans[0], rs[0])
        for p, r in zip(ctx.plans[1:], rs[1:]):
            P.ppd_phit_add(p, r, img)
        return img * (2.0 * g.detach()), None, None   # not differentiable again, like the pieces' nodes


def _transforms_active():
    """Whether a function transform (torch.func) is around.  Torch has no public
    name for it; without this one the answer is the one that is always safe."""
    query = getattr(torch._C, "_are_functorch_transforms_active", None)
    return query is None or bool(query())


def _one_node(plans, x, ys):
    """Whether FidelityFn gives what the composed operations give: constant
    contiguous complex64 data of the plans' sizes without tangents or pending
    conjugation, a real image, no function transform around, and every plan on
    the stream the tensors are on."""
    if (not plans or len(plans) != len(ys) or not (x.is_cuda and x.is_floating_point()) or
            _transforms_active()):
        return False
    here = torch.cuda.current_stream(x.device).cuda_stream
    return all(type(y) is torch.Tensor and y.device == x.device and y.dtype == torch.complex64 and
               not y.requires_grad and not y.is_conj() and not y.is_neg() and y.is_contiguous() and
               y.shape == (p.M,) and p.stream.cuda_stream == here and
               fwAD.unpack_dual(y).tangent is None for p, y in zip(plans, ys))


def data_fidelity(plan, x, y):
    """||Phi x - y||_2^2."""
    if _one_node((plan,), x, (y,)):
        return FidelityFn.apply(x, (plan,), (y,))
    r = phi(plan, x) - y
    return (r.real ** 2 + r.imag ** 2).sum()


def multichannel_fidelity(plans: Sequence, x, ys: Sequence):
    """sum_c ||Phi_c x - y_c||^2 over frequency channels sharing one sky."""
    plans, ys = tuple(plans), tuple(ys)
    if _one_node(plans, x, ys):
        return FidelityFn.apply(x, plans, ys)
    return sum(data_fidelity(p, x, y) for p, y in zip(plans, ys))


class DualUpdateFn(torch.autograd.Function):
    """(v', z') of the data-dual update from g = Theta G F Z x~, v, z and y;
    backward: the library's VJP kernels (the P_B Jacobian per block)."""

    @staticmethod
    def forward(ctx, g, v, z, y, plan, U, eps, n_itr, mu, lam):
        g, v, z, y = (t.detach().contiguous() for t in (g, v, z, y))
        v_out, z_out, zs = P.ppd_dual_update(plan, g, y, U, eps, v, z, n_itr, mu, lam, keep=True)
        ctx.save_for_backward(g, v, z, y, zs)
        ctx.args = (plan, U, eps, n_itr, mu, lam)
        return v_out, z_out

    @staticmethod
    def backward(ctx, gv, gz):
        g, v, z, y, zs = ctx.saved_tensors
        plan, U, eps, n_itr, mu, lam = ctx.args
        gv = None if gv is None else gv.contiguous().to(torch.complex64)
        gz = None if gz is None else gz.contiguous().to(torch.complex128)
        g_g, g_v, g_z, g_y = P.ppd_dual_update_vjp(plan, g, y, U, eps, v, z, n_itr, mu, lam, zs, gv, gz)
        return g_g, g_v, g_z, g_y, None, None, None, None, None, None


class SparsityUpdateFn(torch.autograd.Function):
    """u' = u + lambda (clip(u + c, +-alpha) - u); backward: the clip mask."""

    @staticmethod
    def forward(ctx, u, c, plan, alpha, lam):
        u, c = u.detach().contiguous(), c.detach().contiguous()
        ctx.save_for_backward(u, c)
        ctx.args = (plan, alpha, lam)
        return P.ppd_sparsity_update(plan, u, c, alpha, lam)

    @staticmethod
    def backward(ctx, g):
        u, c = ctx.saved_tensors
        plan, alpha, lam = ctx.args
        g_u, g_c = P.ppd_sparsity_update_vjp(plan, u, c, alpha, lam, g.contiguous().to(torch.float32))
        return g_u, g_c, None, None, None


class PrimalUpdateFn(torch.autograd.Function):
    """(x', x~') of the primal update from x, a = Re Phi^H v', b = Psi u';
    backward: the P_C mask."""

    @staticmethod
    def forward(ctx, x, a, b, plan, tau, eta, zeta, lam):
        x, a, b = (t.detach().contiguous() for t in (x, a, b))
        ctx.save_for_backward(x, a, b)
        ctx.args = (plan, tau, eta, zeta, lam)
        return P.ppd_primal_update(plan, x, a, b, tau, eta, zeta, lam)

    @staticmethod
    def backward(ctx, gx, gxt):
        x, a, b = ctx.saved_tensors
        plan, tau, eta, zeta, lam = ctx.args
        gx = None if gx is None else gx.contiguous().to(torch.float32)
        gxt = None if gxt is None else gxt.contiguous().to(torch.float32)
        g_x, g_a, g_b = P.ppd_primal_update_vjp(plan, x, a, b, tau, eta, zeta, lam, gx, gxt)
        return g_x, g_a, g_b, None, None, None, None, None


def _dense(t, dtype):
    """t as plain memory: contiguous, no pending conjugation or negation.  Most
    are already, and asking costs the host less than the five calls (0.6
    to 1.5 us against 2.8, a dozen tensors an iteration)."""
    if t.requires_grad:
        t = t.detach()
    if t.dtype == dtype and t.is_contiguous() and not t.is_conj() and not t.is_neg():
        return t
    return t.resolve_conj().resolve_neg().contiguous().to(dtype)


class StepFn(torch.autograd.Function):
    """(x', x~', v', u', z') of one iteration from (x, x~, v, u, z, y): one
    library call forward and one backward (its gradients where asked for)."""

    @staticmethod
    def forward(ctx, x, xt, v, u, z, y, plan, U, eps, prm):
        x, v, u, z, y = (_dense(t, t.dtype) for t in (x, v, u, z, y))
        outs, mids = P.ppd_step(plan, x, _dense(xt, torch.float32), v, u, z, y, U, eps, **prm)
        ctx.set_materialize_grads(False)
        # an output that no input with a gradient reaches requires none (x' and x~' are reached by every one)
        _, nxt, nv, nu, nz, ny = ctx.needs_input_grad[:6]
        ctx.mark_non_differentiable(*(() if nxt or nv or nz or ny else (outs[2], outs[4])),
                                    *(() if nxt or nu else (outs[3],)))
        ctx.save_for_backward(x, v, u, z, y, *mids)
        ctx.args = (plan, U, eps, prm)
        return outs

    @staticmethod
    def backward(ctx, *grads):
        x, v, u, z, y, *mids = ctx.saved_tensors
        plan, U, eps, prm = ctx.args
        dts = (torch.float32, torch.float32, torch.complex64, torch.float32, torch.complex128)
        grads = [None if g is None else _dense(g, dt) for g, dt in zip(grads, dts)]
        return P.ppd_step_vjp(plan, x, v, u, z, y, U, eps, mids, grads, ctx.needs_input_grad[:6], **prm) + (None,) * 4


def ppd_iteration(plan, y, U, eps, x, xt, v, u, z, *, tau: float, eta: float, zeta: float = 1.0,
                  lam: float = 1.0, alpha: float = 1e-4, mu: float = 1.0, n_itr: int = 1):
    """One differentiable iteration of Algorithm 3 in the library's data flow
    (plan order): the data-dual update of every block on Theta G F Z x~, the
    sparsity dual update on Psi^H x~, and the primal update on
    Re Phi^H v' and Psi u'; every forward and backward step is a HIP kernel.

    x, xt: (ny, nx) float32; v: (M,) complex64; u: (9, ny, nx) float32;
    z: (M,) complex128; y: (M,) complex64; U: (M,) float64; eps: (d,).
    Returns the new (x, xt, v, u, z)."""
    prm = dict(tau=float(tau), eta=float(eta), zeta=float(zeta), lam=float(lam), alpha=float(alpha), mu=float(mu),
               n_itr=int(n_itr))
    return StepFn.apply(x, xt, v, u, z, y, plan, U, eps, prm)


def unrolled_ppd(plan, block_off, y, U, eps, x0, K: int, *, checkpoint: bool = True, state=None, **params):
    """K differentiable PPD iterations from x = x~ = x0 (v = 0, u = 0, z = y
    unless `state` = (x, xt, v, u, z) is given).  Returns the final x.
    block_off is accepted for compatibility (the plan holds the blocks)."""
    if state is None:
        x, xt = x0, x0
        v = torch.zeros_like(y)
        u = torch.zeros((9,) + tuple(x0.shape), dtype=torch.float32, device=x0.device)
        z = y.to(torch.complex128)
    else:
        x, xt, v, u, z = state
    for _ in range(K):
        if checkpoint:
            x, xt, v, u, z = torch.utils.checkpoint.checkpoint(
                lambda *s: ppd_iteration(plan, y, U, eps, *s, **params),
                x, xt, v, u, z, use_reentrant=False)
        else:
            x, xt, v, u, z = ppd_iteration(plan, y, U, eps, x, xt, v, u, z, **params)
    return x
