"""Couplings in very small or large units and very small amplitudes keep the
precision of FP32: the pieces that the matrix cores multiply hold every bit of
both.  Persistent steps of few and of many trajectories, and coupling kernels
with one launch per step.

Couplings: test_gpu_persist's steps and tolerance against the FP64 oracle, in
units of 2^-122 (24-bit magnitudes that FP32 still holds exactly) and 2^100;
energies scale with the unit.  Amplitudes next to 2^-125: one step against
float64; an update rounds at 4 x 2^-24, and at 2^-149 where it is subnormal:
2-norm within 1e-6."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1807_00699_amd import gd
from paper_1807_00699_amd import inputs as I
from test_gpu_persist import DT, K, TOL, _start

pytestmark = pytest.mark.gpu

ROUTES = [(300, 40, None), (700, 2, None), (300, 40, "1"), (300, 40, "9"), (700, 2, "110"), (700, 2, "100")]


@pytest.mark.parametrize("unit", [-122, 100])
@pytest.mark.parametrize("model", ["ising", "xy"])
@pytest.mark.parametrize("n,R,pin", ROUTES)
def test_couplings_in_any_unit(monkeypatch, n, R, pin, model, unit):
    if pin:
        monkeypatch.setenv("GD_DENSE_CONFIG", pin)
    rng = np.random.default_rng(n)
    m = rng.integers(1 << 20, 1 << 24, (n, n)) * rng.choice([-1, 1], (n, n))
    J = I.sym_from_upper(m.astype(np.float64) * 2.0**-24)
    x0, g0 = _start(model, n, R)
    mdl = gd.GD_ISING if model == "ising" else gd.GD_XY
    E = []
    for u in (0, unit):
        with gd.Solver((J * 2.0**u).astype(np.float32), model=mdl, dt=DT, eps=0.1) as S:
            S.set_state(x0, g0)
            S.run(K)
            x, g, _ = S.state()
            s = S.scale
            S.set_state(x0, g0)
            E.append(S.energy(device_path=True)[0] * 2.0**-u)
    with gd.Solver((J * 2.0**unit).astype(np.float32), model=mdl, dt=DT, eps=0.1, j_scale=s * 2.0**(-unit)) as S:
        S.set_state(x0, g0)     # couplings and their scale in units far apart: no coupling, or beyond FP32
        if unit < 0:
            S.run(K)
            xf, gf, _ = S.state()
            xo, go = O.run(J, x0[:2], g0[:2], model=model, steps=K, dt=DT, eps=0.1, s=1e60)
            assert np.linalg.norm(xf[:2] - xo) <= TOL * np.linalg.norm(xo)
            assert np.linalg.norm(gf[:2] - go) <= TOL * np.linalg.norm(go)
    sub = sorted({0, R // 2, R - 1})
    xo, go = O.run(J, x0[sub], g0[sub], model=model, steps=K, dt=DT, eps=0.1, s=s * 2.0**-unit)
    assert np.linalg.norm(x[sub] - xo) <= TOL * np.linalg.norm(xo)
    assert np.linalg.norm(g[sub] - go) <= TOL * np.linalg.norm(go)
    assert np.allclose(E[0], E[1], rtol=0, atol=1e-6 * np.abs(J).sum())


@pytest.mark.parametrize("coupling", ["pm1", "gauss"])
@pytest.mark.parametrize("model", ["ising", "xy"])
@pytest.mark.parametrize("n,R,pin", ROUTES)
def test_amplitudes_of_any_size(monkeypatch, n, R, pin, model, coupling):
    if pin:
        monkeypatch.setenv("GD_DENSE_CONFIG", pin)
    J = I.dense_pm1(n, 5) if coupling == "pm1" else I.dense_gaussian(n, 5)
    rng = np.random.default_rng([n, R])
    shape = (R, n) if model == "ising" else (R, n, 2)
    x0 = (rng.uniform(0.5, 1.0, shape) * rng.choice([-1.0, 1.0], shape) * 2.0**-124).astype(np.float32)
    with gd.Solver(J, model=gd.GD_ISING if model == "ising" else gd.GD_XY, dt=0.05, eps=0.1) as S:
        S.set_state(x0, np.zeros((R, n), np.float32))
        S.run(1)
        x = S.state()[0].astype(np.float64).reshape(R, n, -1)
        s = S.scale
    p = x0.astype(np.float64).reshape(R, n, -1)
    want = p + 0.05 * np.einsum("ij,rjp->rip", J.astype(np.float64), p) / s
    assert np.linalg.norm((x - want) * 2.0**120) <= 1e-6 * np.linalg.norm(want * 2.0**120)
