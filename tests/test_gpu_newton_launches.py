"""The exact prox by a launch per Newton step at the edges of its chunks (1024
points to half a million, 2048 above): a chunk and one point more, the line
between the two lengths, a long block.  Against the prox in float64 on the host,
to 1e-11 as in test_gpu_newton."""
import numpy as np
import pytest

from oracle import prox as oprox
from gpu_util import announce, host
from test_gpu_newton import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,d", [(1024, 1), (1025, 1), (2049, 2), (524288, 1), (524289, 1), (1_050_001, 3)])
def test_prox_by_launches(M, d):
    announce(f"Newton steps by launches M={M} d={d}")
    P, plan, off, w, y, U, eps, (wd, yd, Ud) = _case(M, d)
    z = host(P.ppd_prox_metric(plan, wd, yd, Ud, eps, n_newton=20))
    for j in range(d):
        s = slice(off[j], off[j + 1])
        ref = oprox.prox_metric_exact(w[s], y[s].astype(np.complex128), eps[j], U[s])
        assert np.linalg.norm(z[s] - ref) <= 1e-11 * np.linalg.norm(ref), j
