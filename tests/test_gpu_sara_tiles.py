"""SARA analysis, synthesis and dual step at the edges of their tiles: images
narrower and lower than a tile, bands of one row or column, every depth, tall
and low analysis tiles, re-weights, and arrays off the 16-byte alignment of
the vector accesses, against the FP64 oracle (the operators' stated parity)."""
import numpy as np
import pytest

from oracle import prox as oprox
from oracle import sara as osara

from gpu_util import announce, assert_op_close, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,nx,levels", [(16, 16, 4), (16, 16, 1), (16, 128, 4), (128, 16, 3), (64, 64, 6),
                                          (32, 256, 2), (256, 512, 3), (512, 256, 5), (1024, 512, 2)])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("weighted", [False, True])
def test_sara_at_tile_edges(ny, nx, levels, shift, weighted):
    P = require_gpu()
    import torch
    announce(f"sara tiles {ny}x{nx} L={levels} shift={shift} W={weighted}")
    plan = P.Plan(nx, ny, np.zeros(1, np.float32), np.zeros(1, np.float32), [0, 1], levels=levels)
    rng = np.random.default_rng(ny * 7 + nx + levels)

    def put(a):   # a contiguous tensor `shift` floats behind an aligned address
        a = np.ascontiguousarray(a, np.float32)
        t = torch.empty(a.size + shift, dtype=torch.float32, device="cuda")[shift:].view(a.shape)
        t.copy_(torch.from_numpy(a))
        return t

    x = rng.standard_normal((ny, nx)).astype(np.float32)
    u = (0.05 * rng.standard_normal((9, ny, nx))).astype(np.float32)
    W = rng.uniform(0.1, 1.0, (9, ny, nx)).astype(np.float32) if weighted else None
    Wd = put(W) if weighted else None
    w64 = W.astype(np.float64) if weighted else 1.0
    c_ref = w64 * osara.analysis(x.astype(np.float64), levels)
    c = P.ppd_sara(plan, P.SARA_ANALYSIS, put(x), out=put(np.zeros_like(u)), W=Wd)
    assert_op_close(host(c), c_ref, what="analysis")
    s = P.ppd_sara(plan, P.SARA_SYNTHESIS, put(u), out=put(np.zeros_like(x)), W=Wd)
    assert_op_close(host(s), osara.synthesis(w64 * u.astype(np.float64), levels), what="synthesis")
    ud, alpha, lam = put(u), 0.05, 0.8
    out = P.ppd_sara(plan, P.SARA_DUAL, put(x), out=put(np.zeros_like(x)), u=ud, alpha=alpha, lam=lam, W=Wd)
    u64 = u.astype(np.float64)
    u_ref = u64 + lam * (oprox.clip_dual(u64 + c_ref, alpha) - u64)
    assert_op_close(host(ud), u_ref, what="dual u")
    assert_op_close(host(out), osara.synthesis(w64 * u_ref, levels), what="dual synthesis")
