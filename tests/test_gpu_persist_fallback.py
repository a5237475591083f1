"""Persistent steps that end early: launches refused by the host side (GD_PERSIST),
launches that give up (GD_PERSIST_WAIT=0: every workgroup, at once) and waits of a
microsecond, which may or may not run out.  The run goes on from the state of the
last good launch, one launch per step, with the statistics of an undisturbed run.

Tolerance against the FP64 oracle: that of test_gpu_persist for the same steps."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1807_00699_amd import gd
from paper_1807_00699_amd import inputs as I
from test_gpu_persist import DT, TOL, _start

pytestmark = pytest.mark.gpu

STEPS, CHECK = 13, 3
CASES = [("ising", 300, 40, False, "pm1"), ("ising", 700, 2, False, "pm1"), ("ising", 1090, 33, False, "gauss"),
         ("xy", 300, 20, True, "gauss")]


def _solver(model, n, rk4, coupling, **kw):
    J = I.dense_pm1(n, 5) if coupling == "pm1" else I.dense_gaussian(n, 5)
    return J, gd.Solver(J, model=gd.GD_ISING if model == "ising" else gd.GD_XY, dt=DT, eps=0.1,
                        integrator=gd.GD_RK4 if rk4 else gd.GD_EULER, **kw)


def _check(S, J, model, rk4, x0, g0, x, g, gave_up=True):
    st = S.stats()
    n, R = J.shape[0], x0.shape[0]
    assert not gave_up or st.kernel_config < 200
    assert st.steps_done == STEPS and st.spin_updates == n * R * STEPS
    steps, trace = S.best_trace()
    assert list(steps) == list(range(CHECK, STEPS + 1, CHECK))
    assert np.all(np.isfinite(trace)) and st.best_energy == trace[-1]
    sub = sorted({0, R // 2, R - 1})
    xo, go = O.run(J, x0[sub], g0[sub], model=model, steps=STEPS, dt=DT, eps=0.1, s=S.scale,
                   integrator=O.RK4 if rk4 else O.EULER)
    assert np.linalg.norm(x[sub] - xo) <= TOL * np.linalg.norm(xo)
    assert np.linalg.norm(g[sub] - go) <= TOL * np.linalg.norm(go)


@pytest.mark.parametrize("model,n,R,rk4,coupling", CASES)
@pytest.mark.parametrize("launches", [0, 1, 2])
def test_refused_launches(monkeypatch, model, n, R, rk4, coupling, launches):
    """After `launches` chunks the steps are those of one launch per step, bit for
    bit, from the state that the launches left."""
    x0, g0 = _start(model, n, R)
    x, g = x0, g0
    if launches:
        J, S = _solver(model, n, rk4, coupling)
        with S:
            S.set_state(x0, g0)
            S.run(CHECK * launches)
            assert S.stats().kernel_config >= 200
            x, g, _ = S.state()
    monkeypatch.setenv("GD_PERSIST", "0")
    J, S = _solver(model, n, rk4, coupling)
    with S:
        S.set_state(x, g)
        S.run(STEPS - CHECK * launches)
        xw, gw, _ = S.state()
    monkeypatch.setenv("GD_PERSIST", str(launches))
    J, S = _solver(model, n, rk4, coupling, check_interval=CHECK)
    with S:
        S.set_state(x0, g0)
        S.run(STEPS)
        x, g, _ = S.state()
        _check(S, J, model, rk4, x0, g0, x, g)
    assert np.array_equal(x, xw) and np.array_equal(g, gw)


@pytest.mark.parametrize("model,n,R,rk4,coupling", CASES)
@pytest.mark.parametrize("wait", ["0", "1"])
@pytest.mark.parametrize("mode", ["deferred", "target", "recorded", "cut"])
def test_waits_that_run_out(monkeypatch, model, n, R, rk4, coupling, mode, wait):
    """Energies of steps that were not taken count for nothing: no best, no
    target, no entry of the trace; and the next set-up starts afresh."""
    monkeypatch.setenv("GD_PERSIST_WAIT", wait)
    monkeypatch.setenv("GD_PERSIST", "1000")
    x0, g0 = _start(model, n, R)
    kw = dict(has_target=1, target_energy=-1e30) if mode == "target" else {}
    J, S = _solver(model, n, rk4, coupling, check_interval=CHECK, **kw)
    with S:
        S.set_state(x0, g0)
        if mode == "recorded":
            gd.gd_set_targets(S.h, [-1e30])
        for m in (5, 1, 7) if mode == "cut" else (STEPS,):
            S.run(m)
        x, g, _ = S.state()
        _check(S, J, model, rk4, x0, g0, x, g, gave_up=wait == "0")
        assert not S.stats().target_reached
        monkeypatch.delenv("GD_PERSIST_WAIT")
        S.set_init(R + 1)
        S.run(CHECK - 1)
        assert S.stats().kernel_config >= 200
