"""The one-node iteration and fidelity as autograd nodes: what requires a
gradient, and what saved-tensor hooks may hand back, as with the pieces."""
import itertools

import pytest

import synth
from gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


def _plan(n=32, M=900, d=2, seed=11):
    P = require_gpu()
    _, wu, wv, off = synth.small_case(n, M, seed=seed, d=d)
    return P.Plan(n, n, wu, wv, off)


def test_iteration_outputs_require_what_the_pieces_require():
    """Each output requires a gradient exactly where the composed pieces' does:
    v', z' with x~, v, z or y, u' with x~ or u, x' and x~' with any."""
    announce("requires_grad of the one-node iteration")
    plan = _plan()
    import torch
    from paper_1701_01748_amd import autograd as A
    M = plan.M
    ins = [torch.rand(32, 32, device="cuda"), torch.rand(32, 32, device="cuda"),
           torch.randn(M, device="cuda", dtype=torch.complex64), 1e-2 * torch.randn(9, 32, 32, device="cuda"),
           torch.randn(M, device="cuda", dtype=torch.complex128), torch.randn(M, device="cuda", dtype=torch.complex64)]
    U = torch.rand(M, device="cuda", dtype=torch.float64) + 0.1
    eps = [5.0, 5.0]
    for need in itertools.product((False, True), repeat=6):
        x, xt, v, u, z, y = (t.clone().requires_grad_(r) for t, r in zip(ins, need))
        out = A.ppd_iteration(plan, y, U, eps, x, xt, v, u, z, tau=0.3, eta=1e-4, n_itr=2)
        v2, z2 = A.DualUpdateFn.apply(A.phi(plan, xt), v, z, y, plan, U, eps, 2, 1.0, 1.0)
        u2 = A.SparsityUpdateFn.apply(u, A.sara_analysis(plan, xt), plan, 1e-4, 1.0)
        x2, xt2 = A.PrimalUpdateFn.apply(x, A.phit(plan, v2), A.sara_synthesis(plan, u2), plan, 0.3, 1e-4, 1.0, 1.0)
        assert [t.requires_grad for t in out] == [t.requires_grad for t in (x2, xt2, v2, u2, z2)], need
        if any(need):   # and backward still runs through what is left
            g = torch.autograd.grad(out[0].sum(), [t for t in (x, xt, v, u, z, y) if t.requires_grad])
            assert all(t is not None for t in g)


@pytest.mark.parametrize("unpack", ["strided", "complex128"])
def test_fidelity_takes_what_saved_tensor_hooks_hand_back(unpack):
    """Hooks may return a saved tensor in another layout or precision, as an
    offloading hook does; the residual is taken as the pieces take a gradient."""
    announce(f"fidelity with saved-tensor hooks, {unpack}")
    plan = _plan()
    import torch
    from paper_1701_01748_amd import autograd as A
    y = torch.randn(plan.M, device="cuda", dtype=torch.complex64)
    x = torch.rand(32, 32, device="cuda").requires_grad_(True)

    def back(h):
        t = torch.stack([h, h], dim=-1).cuda()[..., 0]   # a stride of two
        return t if unpack == "strided" else t.to(torch.complex128 if t.is_complex() else torch.float64)
    ref, = torch.autograd.grad(A.multichannel_fidelity([plan, plan], x, [y, 2 * y]), x)
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t.detach().cpu(), back):
        loss = A.multichannel_fidelity([plan, plan], x, [y, 2 * y])
    assert torch.equal(torch.autograd.grad(loss, x)[0], ref)


def _iteration_grad(plan, hooks):
    import torch
    from paper_1701_01748_amd import autograd as A
    g = torch.Generator(device="cuda").manual_seed(3)
    M = plan.M
    y = torch.randn(M, generator=g, device="cuda", dtype=torch.complex64)
    x = torch.rand(32, 32, generator=g, device="cuda").requires_grad_(True)
    v = 0.1 * torch.randn(M, generator=g, device="cuda", dtype=torch.complex64)
    u = 1e-3 * torch.randn(9, 32, 32, generator=g, device="cuda")
    U = torch.rand(M, generator=g, device="cuda", dtype=torch.float64) + 0.1
    with hooks:
        out = A.ppd_iteration(plan, y, U, [5.0, 5.0], x, x, v, u, y.to(torch.complex128), tau=0.3, eta=1e-4, n_itr=2)
    return torch.autograd.grad(out[0].sum(), x)[0]


@pytest.mark.parametrize("unpack", ["strided", "double", "host"])
def test_iteration_checks_what_saved_tensor_hooks_hand_back(unpack):
    """The iteration's backward pass reads the saved tensors by address: what is
    not plain device memory of the saved type is refused, as by the pieces."""
    announce(f"one-node iteration with saved-tensor hooks, {unpack}")
    plan = _plan()
    import contextlib

    import torch

    def back(h):
        if unpack == "host":
            return h
        if unpack == "double":
            return h.cuda().to(torch.complex128 if h.is_complex() else torch.float64)
        return torch.stack([h, h], dim=-1).cuda()[..., 0]
    ref = _iteration_grad(plan, contextlib.nullcontext())
    assert torch.equal(_iteration_grad(plan, torch.autograd.graph.save_on_cpu()), ref)
    with pytest.raises(ValueError):
        _iteration_grad(plan, torch.autograd.graph.saved_tensors_hooks(lambda t: t.detach().cpu(), back))
