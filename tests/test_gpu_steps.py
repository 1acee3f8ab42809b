"""Algorithm 2 steps and the differentiable dual update at the edges of their
chunks: one point, a chunk and one point more, more blocks than fit a kernel
argument, more chunks than fill the chip, and a block of so many chunks that
its sum is formed by a launch of its own.  Against the same arithmetic in
float64 torch operations: only the order of the norms' sums differs, so
within 1e-12 relative (float32 outputs: half an ulp more, 1e-7)."""
import numpy as np
import pytest

from gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


def _blockwise(off, a):
    import torch
    return torch.stack([a[off[j]:off[j + 1]].sum() for j in range(len(off) - 1)])


def _project(off, y, U, eps, w, z, n):
    import torch
    reps = torch.as_tensor(np.diff(off), device="cuda")
    for _ in range(n):
        q = z - U * (z - w)
        d = q - y
        r = torch.sqrt(_blockwise(off, d.real ** 2 + d.imag ** 2))
        f = torch.where(r > eps, eps / r, torch.ones_like(r))
        z = y + d * torch.repeat_interleave(f, reps)
    return z


def _rel(a, b):
    return float((a - b).abs().norm() / b.abs().norm().clamp_min(1e-300))


@pytest.mark.parametrize("M,d,n_itr", [(1, 1, 1), (512, 1, 2), (513, 2, 3), (70001, 70, 3), (1_200_003, 3, 2),
                                       (8_500_003, 1, 2)])
def test_steps_match_float64(M, d, n_itr):
    P = require_gpu()
    import torch
    from paper_1701_01748_amd import autograd as A
    announce(f"steps M={M} d={d} n_itr={n_itr}")
    g = torch.Generator(device="cuda").manual_seed(M + d)

    def normal(*s):
        return torch.randn(*s, generator=g, device="cuda", dtype=torch.float64)

    def cnormal(s):
        return torch.complex(normal(M), normal(M)) * s
    off = np.round(np.linspace(0, 1, d + 1) ** 1.3 * M).astype(np.int64)
    off[-1] = M
    assert np.all(np.diff(off) > 0)
    y = cnormal(1.0).to(torch.complex64)
    U = torch.rand(M, generator=g, device="cuda", dtype=torch.float64) * 0.9 + 0.05
    y128 = y.to(torch.complex128)
    w, z = y128 + cnormal(0.3), y128 + cnormal(0.1)
    eps = 0.1 * np.sqrt(np.diff(off).astype(np.float64))
    eps[d // 2] *= 100.0   # one block inside its ball
    e = torch.as_tensor(eps, device="cuda")
    ref = _project(off, y128, U, e, w, z, n_itr)
    za = z.clone()
    P.ppd_ellipsoid_proj_noalloc(w, y, U, off, eps, n_itr, 1.0, za)
    assert _rel(za, ref) < 1e-12
    om = ((torch.rand(2, M, generator=g, device="cuda") - 0.5) * 6.0).float().cpu().numpy()
    plan = P.Plan(32, 32, om[0], om[1], off)
    zb = z.clone()
    P.ppd_ellipsoid_proj(plan, w, y, U, eps, n_itr, 1.0, zb)
    assert _rel(zb, ref) < 1e-12
    # forward and VJP of the dual update
    lam = 0.8
    gv = (y128 + cnormal(0.2)).to(torch.complex64)
    v = (U * cnormal(0.1)).to(torch.complex64)
    cv, cz = cnormal(1.0).to(torch.complex64), cnormal(0.5)
    leaves = [t.clone().requires_grad_(True) for t in (gv, v, z, y)]
    v1, z1 = A.DualUpdateFn.apply(*leaves, plan, U, eps, n_itr, 1.0, lam)
    grads = torch.autograd.grad([v1, z1], leaves, [cv, cz])
    leaves64 = [t.to(torch.complex128).clone().requires_grad_(True) for t in (gv, v, z, y)]
    g64, v64, z64, y64 = leaves64
    w64 = v64 / U + g64
    z2 = _project(off, y64, U, e, w64, z64, n_itr)
    v2 = v64 + lam * (U * (w64 - z2) - v64)
    grads64 = torch.autograd.grad([v2, z2], leaves64, [cv.to(torch.complex128), cz])
    assert _rel(z1.detach(), z2.detach()) < 1e-12 and _rel(v1.detach(), v2.detach()) < 1e-7
    for a, b, tol, name in zip(grads, grads64, (1e-7, 1e-7, 1e-11, 1e-7), ("g", "v", "z", "y")):
        assert _rel(a, b) < tol, name
    # without a history the steps run in place of z'
    vn, zn, _ = P.ppd_dual_update(plan, gv, y, U, eps, v, z, n_itr, 1.0, lam)
    assert torch.equal(vn, v1.detach()) and torch.equal(zn, z1.detach())
