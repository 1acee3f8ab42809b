"""The one-node iteration and data fidelity against the same thing composed of
the differentiable pieces: every subset of needed inputs, outputs without a
gradient, one and several channels, and data that only the pieces take (a
pending conjugation, a gradient of its own).  The kernels and their inputs are
the same; sums are formed in another order, so within 1e-6 in norm (a few
float32 ulps), FP64 quantities that only pass through float32 gradients too."""
import pytest

import synth
from gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


def _setup(n=64, M=3000, d=2, seed=7):
    P = require_gpu()
    import torch
    x, wu, wv, off = synth.small_case(n, M, seed=seed, d=d)
    return P, P.Plan(n, n, wu, wv, off), torch.Generator(device="cuda").manual_seed(seed)


def _close(a, b, what):
    assert (a is None) == (b is None), what
    if a is not None:
        assert a.dtype == b.dtype and a.shape == b.shape, what
        scale = float(b.abs().norm()) if b.numel() else 0.0
        assert float((a - b).abs().norm()) <= 1e-6 * scale + 1e-30, what


def _dot(a, b):   # Re <a, b> without a conjugated view, which the pieces do not take as a gradient
    return ((a.real * b.real + a.imag * b.imag) if a.is_complex() else a * b).sum().double()


def _pieces(A, plan, y, U, eps, x, xt, v, u, z, *, tau, eta, zeta, lam, alpha, mu, n_itr):
    g = A.phi(plan, xt)
    v2, z2 = A.DualUpdateFn.apply(g, v, z, y, plan, U, eps, n_itr, mu, lam)
    u2 = A.SparsityUpdateFn.apply(u, A.sara_analysis(plan, xt), plan, alpha, lam)
    x2, xt2 = A.PrimalUpdateFn.apply(x, A.phit(plan, v2), A.sara_synthesis(plan, u2), plan, tau, eta, zeta, lam)
    return x2, xt2, v2, u2, z2


@pytest.mark.parametrize("outs", [(0,), (1,), (2,), (3,), (4,), (0, 3), (2, 3), (1, 4), (0, 1, 2, 3, 4)])
def test_iteration_matches_its_pieces(outs):
    P, plan, g = _setup()
    import torch
    from paper_1701_01748_amd import autograd as A
    announce(f"one-node iteration, gradients of outputs {outs}")
    N, M = plan.N, plan.M

    def rand(*s, dtype=torch.float32):
        return torch.randn(*s, generator=g, device="cuda", dtype=dtype)
    ins = [rand(64, 64), rand(64, 64), rand(M, dtype=torch.complex64), 1e-2 * rand(9, 64, 64),
           rand(M, dtype=torch.complex128), rand(M, dtype=torch.complex64)]
    U = torch.rand(M, generator=g, device="cuda", dtype=torch.float64) * 0.9 + 0.05
    eps = [20.0, 1e3]
    prm = dict(tau=0.3, eta=0.2, zeta=0.9, lam=0.8, alpha=1e-2, mu=0.7, n_itr=2)
    cot = None
    for need in [(True,) * 6] + [tuple(j == k for j in range(6)) for k in range(6)]:
        got = []
        for f in (lambda x, xt, v, u, z, y: A.ppd_iteration(plan, y, U, eps, x, xt, v, u, z, **prm),
                  lambda x, xt, v, u, z, y: _pieces(A, plan, y, U, eps, x, xt, v, u, z, **prm)):
            leaves = [t.clone().requires_grad_(r) for t, r in zip(ins, need)]
            res = f(*leaves)
            cot = cot or [torch.randn(t.shape, generator=g, device="cuda", dtype=t.dtype) for t in res]
            loss = sum(_dot(res[k], cot[k]) for k in outs)
            gr = torch.autograd.grad(loss, [t for t in leaves if t.requires_grad], allow_unused=True) \
                if loss.requires_grad else [None] * sum(need)
            got.append(([t.detach() for t in res], gr))
        for k, (a, b) in enumerate(zip(got[0][0], got[1][0])):
            _close(a, b, f"output {k}")
        for k, (a, b) in enumerate(zip(got[0][1], got[1][1])):
            if b is None or a is None:   # an output that an input does not reach: nothing, or zeros
                assert all(t is None or not bool(t.abs().any()) for t in (a, b)), f"gradient {k}, need {need}"
            else:
                _close(a, b, f"gradient {k}, need {need}")


@pytest.mark.parametrize("data", ["plain", "conj", "grad", "float64 image"])
@pytest.mark.parametrize("C", [1, 3])
def test_fidelity_matches_its_pieces(C, data):
    P, _, g = _setup()
    import torch
    from paper_1701_01748_amd import autograd as A
    announce(f"one-node fidelity C={C} {data}")
    plans = [_setup(M=2000 + 1777 * c, seed=20 + c)[1] for c in range(C)]
    ys = [torch.randn(p.M, generator=g, device="cuda", dtype=torch.complex64) for p in plans]
    x = torch.randn(64, 64, generator=g, device="cuda", dtype=torch.float64 if "float64" in data else torch.float32)
    if data == "conj":
        ys = [y.conj() for y in ys]
    if data == "grad":
        ys[-1].requires_grad_(True)
    x.requires_grad_(True)
    loss = A.multichannel_fidelity(plans, x, ys)
    rs = [A.phi(p, x) - y for p, y in zip(plans, ys)]
    ref = sum((r.real ** 2 + r.imag ** 2).sum() for r in rs)
    assert loss.dtype == ref.dtype and loss.shape == ref.shape
    _close(loss.detach(), ref.detach(), "loss")
    leaves = [x] + [y for y in ys if y.requires_grad]
    for a, b in zip(torch.autograd.grad(3.0 * loss, leaves), torch.autograd.grad(3.0 * ref, leaves)):
        _close(a, b, "gradient")
