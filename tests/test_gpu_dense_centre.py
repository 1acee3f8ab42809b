"""Gridding where a few tiles hold most points, so that their items' regions are
added up in groups before the fold: on either side of the lines (more than 128
items in a tile of 8 x 8, 32 in larger ones), against the FP64 oracle to the
operators' stated parity; and paired launches bitwise as separate ones."""
import numpy as np
import pytest

from oracle import nufft as onf
from gpu_util import announce, assert_op_close, dev, host, require_gpu

pytestmark = pytest.mark.gpu


def _coverage(M, seed, spread=1e-3):
    """Most points within a cell of the centre and of a wrapped corner, the rest anywhere."""
    rng = np.random.default_rng(seed)
    w = spread * rng.standard_normal((2, M)) + 1e-2
    w[:, M // 3:M // 2] += 3.12
    w[:, ::37] = rng.uniform(-3.1, 3.1, w[:, ::37].shape)
    return np.clip(w, -3.14, 3.14).astype(np.float32)


@pytest.mark.parametrize("M,tile,chunk", [(6000, 8, 64), (24000, 8, 64), (40000, 8, 128), (4000, 16, 64), (9000, 16, 64),
                                          (9000, 32, 64), (9000, 64, 64)])
def test_phit_of_a_dense_centre(M, tile, chunk):
    P = require_gpu()
    import torch
    announce(f"dense centre M={M} tile={tile} chunk={chunk}")
    wu, wv = _coverage(M, M + tile)
    plan = P.Plan(64, 32, wu, wv, np.array([0, M // 4, M], np.int64), tile=tile, chunk=chunk)
    rng = np.random.default_rng(3)
    v = (rng.standard_normal(M) + 1j * rng.standard_normal(M)).astype(np.complex64)
    got = host(P.ppd_phit(plan, dev(v, torch.complex64), order=P.ORDER_USER))
    assert_op_close(got, onf.Nufft(wu, wv, 32, 64).phit(v.astype(np.complex128)), what="phit")


@pytest.mark.parametrize("levels", [1, 3, 4])
@pytest.mark.parametrize("weighted", [False, True])
def test_paired_launches_of_a_dense_centre(levels, weighted):
    P = require_gpu()
    import torch
    announce(f"dense centre, paired, levels={levels} weighted={weighted}")
    M = 30000
    wu, wv = _coverage(M, 5)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        plan = P.Plan(64, 64, wu, wv, np.array([0, M // 4, M], np.int64), chunk=64, levels=levels, stream=stream)
        g = torch.Generator(device="cuda").manual_seed(1)
        y = P.ppd_phi(plan, torch.rand(64, 64, generator=g, device="cuda"))
        U = torch.rand(M, generator=g, device="cuda", dtype=torch.float64) * 0.9 + 0.05
        W = torch.rand(9, 64, 64, generator=g, device="cuda") if weighted else None
        eps = np.array([0.1, 0.2]) * float(y.abs().square().sum().sqrt())
        got = []
        for timed, graph in ((True, False), (False, False), (False, True)):
            st = P.PPDState(plan, y)
            plan.timing(timed)
            P.ppd_iterate(plan, st, y, U, eps, 3, eta=1e-8, stats=False, use_graph=graph, W=W)
            assert plan.forms()["paired"] is not timed
            got.append([t.clone() for t in (st.x, st.xt, st.v, st.u, st.z)])
        plan.timing(False)
    assert bool(got[0][0].any())
    for other in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], other))
