"""The measurement operator on the half spectrum: every transform length along
rows and columns, and visibilities at the edges of the kept half plane
(around the v axis on either side of the mirroring rule, at the Nyquist
column, at the wrapped grid rows), for every tile size, against the FP64
oracle.  The bound is the operators' stated parity."""
import numpy as np
import pytest

from oracle import nufft as onf

from gpu_util import announce, assert_op_close, dev, host, require_gpu

pytestmark = pytest.mark.gpu


def _edge_coverage(ny, nx, seed):
    """Grid coordinates at and beside each edge of the kept half plane, both
    signs, and random points; (wu, wv) float32."""
    rng = np.random.default_rng(seed)
    lo = float(np.nextafter(np.float32(np.pi), np.float32(0)))

    def axis(K):
        t = np.array([-K / 2, -K / 2 + 0.5, -6.0, -5.5, -5.0, -4.999, -3.0, -0.5, 0.0, 0.5, 2.999, 3.0, 5.0, 5.5,
                      K / 2 - 4.5, K / 2 - 3.0, K / 2 - 0.5, K / 2])
        return np.clip(t * 2 * np.pi / K, -lo, lo)
    au, av = axis(2 * nx), axis(2 * ny)
    gu, gv = (a.ravel() for a in np.meshgrid(au, av))
    ru, rv = rng.uniform(-lo, lo, (2, 301))
    return np.concatenate([gu, ru]).astype(np.float32), np.concatenate([gv, rv]).astype(np.float32)


@pytest.mark.parametrize("ny,nx,tile", [(16, 2048, 8), (2048, 16, 8), (32, 1024, 8), (1024, 32, 8), (512, 16, 8),
                                        (16, 512, 8), (256, 64, 8), (64, 256, 8), (128, 16, 8), (16, 128, 8),
                                        (32, 32, 8), (16, 16, 16), (16, 16, 32), (32, 16, 64), (64, 32, 64),
                                        (64, 64, 16), (32, 128, 32)])
def test_operator_at_the_half_plane_edges(ny, nx, tile):
    P = require_gpu()
    import torch
    announce(f"half plane {ny}x{nx} tile={tile}")
    wu, wv = _edge_coverage(ny, nx, seed=ny + nx + tile)
    M = wu.size
    rng = np.random.default_rng(M + nx)
    plan = P.Plan(nx, ny, wu, wv, np.array([0, M // 3, M], np.int64), tile=tile)
    op = onf.Nufft(wu, wv, ny, nx)
    x = rng.standard_normal((ny, nx)).astype(np.float32)
    y = host(P.ppd_phi(plan, dev(x, torch.float32), order=P.ORDER_USER))
    assert_op_close(y, op.phi(x.astype(np.float64)), what="phi")
    v = (rng.standard_normal(M) + 1j * rng.standard_normal(M)).astype(np.complex64)
    xg = host(P.ppd_phit(plan, dev(v, torch.complex64), order=P.ORDER_USER))
    assert_op_close(xg, op.phit(v.astype(np.complex128)), what="phit")
