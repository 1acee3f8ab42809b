"""The caller's order with so many blocks that it takes a permutation pass of
its own, on either side of the lines (8192 blocks, 524288 points): the same
values as in plan order, permuted, and the same image; and the pass is counted."""
import numpy as np
import pytest

from gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,d,apart", [(524289, 8193, True), (524289, 8192, False), (524288, 8193, False),
                                       (700001, 30000, True)])
def test_user_order_is_the_permuted_plan_order(M, d, apart):
    P = require_gpu()
    import torch
    announce(f"user order M={M} d={d}")
    rng = np.random.default_rng(d)
    wu, wv = rng.uniform(-3.1, 3.1, (2, M)).astype(np.float32)
    plan = P.Plan(64, 128, wu, wv, np.round(np.linspace(0, M, d + 1)).astype(np.int64))
    g = torch.Generator(device="cuda").manual_seed(d)
    x = torch.randn(128, 64, generator=g, device="cuda")
    v = torch.randn(M, generator=g, device="cuda", dtype=torch.complex64)
    y = plan.permute(P.PLAN_TO_USER, P.ppd_phi(plan, x))
    img = P.ppd_phit(plan, plan.permute(P.USER_TO_PLAN, v))
    plan.timing(True)
    keep = v.clone()
    assert torch.equal(P.ppd_phi(plan, x, order=P.ORDER_USER), y)
    assert torch.equal(P.ppd_phit(plan, v, order=P.ORDER_USER), img) and torch.equal(v, keep)
    assert plan.timing_read().get("permute", (0, 0.0))[0] == (2 if apart else 0)
    plan.timing(False)
