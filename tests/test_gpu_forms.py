"""Which form an iteration takes, asserted case by case (ppd_plan_get_forms):
the tests that compare the forms' results hold whatever form runs, so they
would not notice one that is never taken.  The cases are theirs."""
import numpy as np
import pytest

import synth
from gpu_util import announce, dev, host, require_gpu

pytestmark = pytest.mark.gpu


def _case(M, d, n=64, nx=None, **plan_kw):
    P = require_gpu()
    import torch
    rng = np.random.default_rng(M + d)
    _, wu, wv, off = synth.small_case(n, M, seed=5, nx=nx, d=d)
    stream = torch.cuda.Stream()
    plan = P.Plan(nx or n, n, wu, wv, off, stream=stream, **plan_kw)
    y = dev((rng.standard_normal(M) + 1j * rng.standard_normal(M)).astype(np.complex64), torch.complex64)
    U = dev(rng.uniform(0.02, 1.0, M), torch.float64)
    eps = 0.1 * np.sqrt(np.diff(off).astype(np.float64))
    torch.cuda.synchronize()
    return P, torch, stream, plan, y, U, eps


def _forms(case, n_iter=1, **kw):
    """(forms, x, z) after n_iter iterations from the start state."""
    P, torch, stream, plan, y, U, eps = case
    with torch.cuda.stream(stream):
        st = P.PPDState(plan, y)
        P.ppd_iterate(plan, st, y, U, eps, n_iter, eta=1e-4, stats=False, **kw)
        f = plan.forms()
    return f, host(st.x), host(st.z)


# image rows, columns, points, blocks, Algorithm 2 steps (0: exact prox), levels; paired eager, paired replayed
@pytest.mark.parametrize("n,nx,M,d,n_itr,levels,eager,replayed", [
    (16, 16, 300, 1, 1, 3, True, True), (32, 64, 2000, 2, 2, 1, True, True), (64, 32, 2001, 1, 1, 4, True, True),
    (64, 64, 4096, 2, 3, 3, True, True), (128, 128, 60000, 3, 1, 3, True, True),
    (128, 128, 20000, 2, 0, 4, True, True), (128, 128, 40000, 2, 0, 4, True, False),
    (64, 64, 9000, 5, 0, 2, True, True), (64, 64, 4096, 2, 0, 3, True, True),
    (256, 256, 65536, 4, 5, 3, True, False), (512, 64, 30000, 2, 1, 3, True, True),
    (64, 64, 4096, 2, 1, 5, False, False), (512, 512, 200000, 2, 1, 3, False, False)])
def test_pairing(n, nx, M, d, n_itr, levels, eager, replayed):
    announce(f"pairing {n}x{nx} M={M} d={d} n_itr={n_itr} levels={levels}")
    case = _case(M, d, n, nx, levels=levels)
    P, plan = case[0], case[3]
    kw = dict(n_itr=n_itr) if n_itr else dict(prox=P.PROX_EXACT)
    print(plan.info.n_chunks, "items", flush=True)
    assert _forms(case, **kw)[0]["paired"] is eager
    assert _forms(case, use_graph=True, **kw)[0]["paired"] is replayed
    plan.timing(True)   # separate launches, each timed
    assert _forms(case, **kw)[0]["paired"] is False


@pytest.mark.parametrize("M,d,one", [(1, 1, True), (512, 1, True), (513, 2, True), (4000, 4, True), (4000, 40, False),
                                     (131072, 3, True), (131073, 3, True), (200003, 8, True), (524289, 5, True)])
def test_newton_steps_in_one_launch(M, d, one):
    announce(f"Newton form M={M} d={d}")
    case = _case(M, d)
    P = case[0]
    kw = dict(prox=P.PROX_EXACT)
    ref, xr, zr = _forms(case, persistent=P.PERSIST_OFF, **kw)
    assert ref["one_launch"] is False and ref["solved_alone"] == 0
    f, x, z = _forms(case, **kw)
    assert f["one_launch"] is one and f["solved_alone"] == 0
    assert np.linalg.norm(z - zr) <= 1e-11 * np.linalg.norm(zr)


@pytest.mark.parametrize("M,d", [(131072, 3), (200003, 8)])   # 256 and 196 workgroups
def test_newton_solve_by_one_workgroup(M, d):
    announce(f"Newton solve by one workgroup M={M} d={d}")
    case = _case(M, d)
    P = case[0]
    kw = dict(prox=P.PROX_EXACT)
    _, _, zr = _forms(case, persistent=P.PERSIST_OFF, **kw)
    alone = 0
    for lim in (1, 1, 1, 1, 0):   # one poll is too few in all but a rare launch; then as it was left
        f, _, z = _forms(case, spin_limit=lim, **kw)
        assert f["one_launch"] and (f["solved_alone"] == alone or lim == 1)
        alone = f["solved_alone"]
        assert np.linalg.norm(z - zr) <= 1e-11 * np.linalg.norm(zr)
    assert 1 <= alone <= 4


def test_timers_leave_replayed_iterations_alone():
    """Timers do not reach captured launches: a graph captured while they are
    on is the same one, which later calls with the same arguments replay."""
    announce("pairing of a graph captured with the timers on")
    case = _case(4096, 2)
    P, torch, stream, plan, y, U, eps = case
    with torch.cuda.stream(stream):
        it = P.Iteration(plan, P.PPDState(plan, y), y, U, eps, eta=1e-4, use_graph=True)
        for on in (True, False, True):
            plan.timing(on)
            it.run(2)
            assert plan.forms()["paired"], on


def test_newton_steps_leave_room_for_other_launches():
    """One launch only where four of it fit the device; a plan of a million
    points takes a launch per step, which waits for nothing."""
    announce("Newton form at 1000000 points")
    case = _case(1_000_000, 5)
    assert _forms(case, prox=case[0].PROX_EXACT)[0]["one_launch"] is False


@pytest.mark.parametrize("n_newton", [1, 7])
def test_prox_metric_waits_for_nothing(n_newton):
    """ppd_prox_metric has no argument that turns waits off: a launch per step."""
    announce(f"ppd_prox_metric launches, {n_newton} steps")
    case = _case(5000, 2)
    P, torch, stream, plan, y, U, eps = case
    with torch.cuda.stream(stream):
        plan.timing(True)
        P.ppd_prox_metric(plan, y.to(torch.complex128), y, U, eps, n_newton=n_newton)
        assert plan.timing_read()["subiter"][0] == n_newton
        plan.timing(False)


@pytest.mark.parametrize("M", [65536, 131072, 200003, 327680, 327681, 400000, 500000, 1300000])
def test_algorithm2_launches_fit_beside_each_other(M):
    """Fewer points per thread must not cost room: four launches of a plan (as
    many as a process's hardware queues run at once) fit the device wherever
    they do with the longest chunks, 3072 points and 512 workgroups."""
    announce(f"room for Algorithm 2 launches M={M}")
    assert _case(M, 4)[3].forms()["beside"] >= min(4, 512 // -(-M // 3072)) >= 1


@pytest.mark.parametrize("M,d", [(65536, 4), (131072, 1), (200003, 8), (500000, 5)])   # 2, 2, 4, 12 points per thread
@pytest.mark.parametrize("n_itr", [3, 5])
@pytest.mark.parametrize("masked", [False, True])
def test_middle_steps_by_one_workgroup(M, d, n_itr, masked):
    """A wait that gives up costs time only: the last workgroup forms the steps
    (the bounds are the Newton launch's: the sums' order moves r by a few ulps)."""
    announce(f"Algorithm 2 steps by one workgroup M={M} d={d} n_itr={n_itr} masked={masked}")
    case = _case(M, d)
    P, torch, stream, plan, y, U, eps = case
    kw = dict(n_itr=n_itr)
    if masked:
        kw["block_active"] = torch.tensor([k != 0 or d == 1 for k in range(d)], device="cuda").to(torch.uint8)
        torch.cuda.synchronize()
    _, xr, zr = _forms(case, persistent=P.PERSIST_OFF, **kw)
    gave_up = 0
    for lim in (1, 1, 1, 1, 0):   # one poll is too few in all but a rare launch; then as it was left
        f, x, z = _forms(case, spin_limit=lim, **kw)
        assert f["one_launch"] and (f["solved_alone"] == gave_up or lim == 1)
        gave_up = f["solved_alone"]
        assert np.linalg.norm(z - zr) <= 1e-11 * np.linalg.norm(zr)
        assert np.linalg.norm(x - xr) <= 1e-6 * np.linalg.norm(xr)
    assert 1 <= gave_up <= 4
    # the given limit that was reached is still reported, once
    with torch.cuda.stream(stream):
        st = P.PPDState(plan, y)
        with pytest.raises(P.PPDError) as err:
            P.ppd_iterate(plan, st, y, U, eps, 1, eta=1e-4, **kw)
        assert err.value.status == P.PPD_EDEVICE and "gave up" in str(err.value)
        P.ppd_iterate(plan, st, y, U, eps, 1, eta=1e-4, **kw)
