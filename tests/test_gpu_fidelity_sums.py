"""The data fidelity's value where its sum has many terms: many blocks (items of
up to 64 segments of a point or two), one block, shared items, several waves
per item and the larger tiles, and several channels.  The squares are of
float64 differences, the stored residual is those rounded to float32 (2^-24 each,
2^-23 in a square): against the stored ones' squares in float64, 2e-7."""
import numpy as np
import pytest

import synth
from gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,M,d,tile", [(16, 1, 1, 8), (32, 65, 65, 8), (64, 5000, 1, 8), (64, 5000, 700, 8),
                                        (256, 300000, 20000, 8), (256, 700000, 3, 8), (64, 20000, 9000, 16),
                                        (64, 20000, 5, 32), (128, 20000, 300, 64)])
def test_fidelity_value(n, M, d, tile):
    P = require_gpu()
    import torch
    from paper_1701_01748_amd import autograd as A
    announce(f"fidelity value {n}^2 M={M} d={d} tile={tile}")
    _, wu, wv, _ = synth.small_case(n, M, seed=4)
    plan = P.Plan(n, n, wu, wv, np.round(np.linspace(0, M, d + 1)).astype(np.int64), tile=tile)
    g = torch.Generator(device="cuda").manual_seed(M)
    x = torch.rand(n, n, generator=g, device="cuda")
    y = torch.randn(M, generator=g, device="cuda", dtype=torch.complex64)
    r = A.phi(plan, x) - y
    ref = float((r.real.double() ** 2 + r.imag.double() ** 2).sum())
    acc = torch.empty(1, dtype=torch.float64, device="cuda")
    loss = torch.empty((), dtype=torch.float32, device="cuda")
    r1 = P.ppd_fidelity(plan, x, y, acc, loss, False)
    assert torch.equal(r1, r)
    assert abs(float(acc) - ref) <= 2e-7 * ref and abs(float(loss) - float(acc)) <= 1e-7 * ref
    first = float(acc)
    P.ppd_fidelity(plan, x, y, acc, loss, True)   # a second channel is added
    assert abs(float(acc) - 2.0 * first) <= 1e-12 * first   # in another order
    assert float(A.multichannel_fidelity([plan, plan], x, [y, y])) == float(loss)
