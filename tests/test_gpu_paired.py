"""Small problems run SARA's launches inside the data path's; with the plan's
per-kernel timers on, every launch is its own.  Both do the same arithmetic in
the same order, so the iterates must agree bitwise: square and oblong images at
the tile sizes' edges, one and several Algorithm 2 steps, weights, inactive
blocks and bases, eager and replayed."""
import pytest

import synth
from gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nx,M,d,n_itr,levels", [(16, 16, 300, 1, 1, 3), (32, 64, 2000, 2, 2, 1),
                                                   (64, 32, 2001, 1, 1, 4), (64, 64, 4096, 2, 3, 3),
                                                   (128, 128, 60000, 3, 1, 3), (128, 128, 20000, 2, 0, 4),
                                                   (64, 64, 9000, 5, 0, 2), (64, 64, 4096, 2, 0, 3),
                                                   (128, 64, 9000, 3, 1, 2), (256, 256, 65536, 4, 5, 3),
                                                   (512, 64, 30000, 2, 1, 3)])
@pytest.mark.parametrize("masked", [False, True])
def test_paired_launches_match_separate_ones(n, nx, M, d, n_itr, levels, masked):
    P = require_gpu()
    import torch
    announce(f"paired launches n={n} nx={nx} M={M} d={d} n_itr={n_itr} levels={levels} masked={masked}")
    x, wu, wv, off = synth.small_case(n, M, seed=3, nx=nx, d=d)
    g = torch.Generator(device="cuda").manual_seed(n + M)

    def rand(*s, dtype=torch.float32):
        return torch.randn(*s, generator=g, device="cuda", dtype=dtype)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        plan = P.Plan(nx, n, wu, wv, off, levels=levels, stream=stream)
        sky = torch.as_tensor(x, dtype=torch.float32, device="cuda")
        y = P.ppd_phi(plan, sky)
        y += 0.05 * y.abs().square().mean().sqrt() * rand(M, dtype=torch.complex64)
        eps = [0.1 * float(y[a:b].abs().square().sum().sqrt()) for a, b in zip(off[:-1], off[1:])]
        U = torch.rand(M, generator=g, device="cuda", dtype=torch.float64) * 0.9 + 0.05
        eta = 1.0 / P.ppd_op_norm(plan, U, sky + 1.0, 10, 1e-2)[0]
        kw = dict(n_itr=n_itr) if n_itr else dict(prox=P.PROX_EXACT)   # 0: the exact prox
        kw.update(eta=eta, alpha=1e-3 * float(sky.abs().max()))
        if masked:
            kw.update(W=torch.rand(9, plan.ny, plan.nx, generator=g, device="cuda") + 0.5,
                      block_active=torch.tensor([k != 0 or d == 1 for k in range(d)], device="cuda").to(torch.uint8),
                      basis_active=torch.tensor([k % 3 != 1 for k in range(9)], device="cuda").to(torch.uint8))
        got = {}
        for name, timed, graph in (("separate", True, False), ("paired", False, False), ("replayed", False, True)):
            st = P.PPDState(plan, y)
            plan.timing(timed)
            for _ in range(3):
                P.ppd_iterate(plan, st, y, U, eps, 2, use_graph=graph, **kw)
            stream.synchronize()
            got[name] = [t.clone() for t in (st.x, st.xt, st.v, st.u, st.z)]
        plan.timing(False)
    ref = got.pop("separate")
    assert bool(ref[0].any()) and bool(ref[3].any())
    for name, ts in got.items():
        for k, (a, b) in enumerate(zip(ts, ref)):
            assert torch.equal(a, b), (name, "x xt v u z".split()[k])
