"""The exact prox's Newton steps as one launch: chunks of points per workgroup
at their edges (the three chunk lengths, a single point, a ragged last
workgroup), blocks inside their ball, and waits that give up at once, after
which one workgroup solves alone.  Against the prox in float64 on the host and
against the launches step by step.  The sums' order moves r by a few ulps,
and nu by no more than that times (max U + nu), so z agrees to 1e-11."""
import numpy as np
import pytest

import synth
from oracle import prox as oprox
from gpu_util import announce, dev, host, require_gpu

pytestmark = pytest.mark.gpu


def _case(M, d):
    P = require_gpu()
    import torch
    rng = np.random.default_rng(M + d)
    _, wu, wv, off = synth.small_case(64, M, seed=5, d=d)
    plan = P.Plan(64, 64, wu, wv, off)

    def cn(s):
        return s * (rng.standard_normal(M) + 1j * rng.standard_normal(M))
    y = cn(1.0).astype(np.complex64)
    U = rng.uniform(0.02, 1.0, M)
    w = y.astype(np.complex128) + cn(0.3)
    eps = 0.1 * np.sqrt(np.diff(off).astype(np.float64))
    if d > 1:
        eps[d // 2] *= 100.0   # one block inside its ball
    return P, plan, off, w, y, U, eps, (dev(w, torch.complex128), dev(y, torch.complex64), dev(U, torch.float64))


@pytest.mark.parametrize("M,d", [(1, 1), (512, 1), (513, 2), (4000, 4), (131072, 3), (131073, 3), (524289, 5)])
def test_prox_matches_host(M, d):
    announce(f"one-launch Newton steps M={M} d={d}")
    P, plan, off, w, y, U, eps, (wd, yd, Ud) = _case(M, d)
    for _ in range(2):   # the second finds the slots as the first left them
        z = host(P.ppd_prox_metric(plan, wd, yd, Ud, eps, n_newton=40))
        for j in range(d):
            s = slice(off[j], off[j + 1])
            ref = oprox.prox_metric_exact(w[s], y[s].astype(np.complex128), eps[j], U[s])
            assert np.linalg.norm(z[s] - ref) <= 1e-11 * np.linalg.norm(ref), j


@pytest.mark.parametrize("M,d", [(513, 2), (4000, 4), (131073, 3)])
@pytest.mark.parametrize("n_newton", [1, 3, 12])
def test_iteration_matches_launches_also_after_a_give_up(M, d, n_newton):
    announce(f"one-launch Newton steps in an iteration M={M} d={d} n_newton={n_newton}")
    P, plan, off, _, y, U, eps, (wd, yd, Ud) = _case(M, d)
    got = {}
    for name, kw in (("launches", dict(persistent=P.PERSIST_OFF)), ("one", {}), ("give-up", dict(spin_limit=1)),
                     ("again", {})):
        st = P.PPDState(plan, yd)
        P.ppd_iterate(plan, st, yd, Ud, eps, 1, eta=1e-4, prox=P.PROX_EXACT, n_newton=n_newton, **kw)
        got[name] = (host(st.z), host(st.v))
    ref = got.pop("launches")
    for name, (z, v) in got.items():
        assert np.linalg.norm(z - ref[0]) <= 1e-11 * np.linalg.norm(ref[0]), name
        assert np.linalg.norm(v - ref[1]) <= 1e-6 * np.linalg.norm(ref[1]), name
    assert np.array_equal(got["one"][0], got["again"][0])
