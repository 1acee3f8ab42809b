"""Paired launches only up to 1024 blocks, on either side of the line, and the
same iterates bitwise as separate launches with the timers on."""
import numpy as np
import pytest

import synth
from gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,paired", [(1023, True), (1024, True), (1025, False), (4096, False)])
@pytest.mark.parametrize("graph", [False, True])
def test_pairing_by_blocks(d, paired, graph):
    P = require_gpu()
    import torch
    announce(f"pairing with {d} blocks graph={graph}")
    M, n = 4096, 64
    _, wu, wv, _ = synth.small_case(n, M, seed=9)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        plan = P.Plan(n, n, wu, wv, np.round(np.linspace(0, M, d + 1)).astype(np.int64), stream=stream)
        g = torch.Generator(device="cuda").manual_seed(d)
        y = P.ppd_phi(plan, torch.rand(n, n, generator=g, device="cuda"))
        U = torch.rand(M, generator=g, device="cuda", dtype=torch.float64) * 0.9 + 0.05
        eps = np.full(d, 0.1)
        got = []
        for timed in (True, False):
            st = P.PPDState(plan, y)
            plan.timing(timed)
            P.ppd_iterate(plan, st, y, U, eps, 3, eta=1e-5, stats=False, use_graph=graph and not timed)
            assert plan.forms()["paired"] is (paired and not timed)
            got.append([t.clone() for t in (st.x, st.xt, st.v, st.u, st.z)])
        plan.timing(False)
    assert bool(got[0][0].any()) and all(torch.equal(a, b) for a, b in zip(*got))
