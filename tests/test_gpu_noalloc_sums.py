"""ppd_ellipsoid_proj_noalloc where a block has more chunks than its workgroups
add up themselves (4096 of 8192 points): the block's sum is formed by a launch
of its own, with the block tables as kernel arguments (to 64 blocks) and in the
fixed array.  Against the same arithmetic in float64 torch operations: only the
order of the norms' sums differs, so within 1e-12 relative."""
import numpy as np
import pytest

from gpu_util import announce, require_gpu
from test_gpu_steps import _project, _rel

pytestmark = pytest.mark.gpu

OWN_SUM = 4096 * 8192   # points of the longest block without a launch for its sum


@pytest.mark.parametrize("big,d", [(OWN_SUM, 2), (OWN_SUM + 1, 2), (OWN_SUM + 20_001, 64), (OWN_SUM + 20_001, 65)])
def test_noalloc_block_sums_in_a_launch(big, d):
    P = require_gpu()
    import torch
    announce(f"noalloc sums block of {big} of {d}")
    sizes = np.full(d, 701, dtype=np.int64)
    sizes[d // 2] = big
    off = np.concatenate([[0], np.cumsum(sizes)])
    M = int(off[-1])
    g = torch.Generator(device="cuda").manual_seed(d)

    def cnormal(s):
        return s * torch.randn(M, generator=g, device="cuda", dtype=torch.complex128)
    y = cnormal(1.0).to(torch.complex64)
    y128 = y.to(torch.complex128)
    U = torch.rand(M, generator=g, device="cuda", dtype=torch.float64) * 0.9 + 0.05
    w, z = y128 + cnormal(0.3), y128 + cnormal(0.1)
    eps = 0.1 * np.sqrt(sizes.astype(np.float64))
    eps[0] *= 100.0   # one block inside its ball
    ref = _project(off, y128, U, torch.as_tensor(eps, device="cuda"), w, z, 3)
    P.ppd_ellipsoid_proj_noalloc(w, y, U, off, eps, 3, 1.0, z)
    # block by block: a small one's norm is lost in the whole's
    assert max(_rel(z[a:b], ref[a:b]) for a, b in zip(off[:-1], off[1:])) < 1e-12
