"""Reduced-precision coupling kernels on FP8-stored couplings (gd_split.h,
variant ids from 14 on): the same operands, products and order of the sums as
variants 4-13, so the same bits; and, at sizes those do not tile, the one-step
bound derived in test_gpu_lowprec."""
import numpy as np
import pytest

from paper_1807_00699_amd import gd
from paper_1807_00699_amd import inputs as I
from test_gpu_lowprec import _one_step_check

pytestmark = pytest.mark.gpu

IDS = range(14, 19)


def _run(J, x, gam, prec, model, integrator, steps=3):
    with gd.Solver(J, model=model, precision=prec, dt=0.03, eps=0.1, integrator=integrator) as S:
        S.set_state(x, gam)
        S.run(steps)
        E, best = S.energy()
        Ed, bd = S.energy(device_path=True)
        assert S.stats().diverged == 0
        return S.state()[:2] + (E, Ed)


@pytest.mark.parametrize("prec", [gd.GD_PREC_BF16, gd.GD_PREC_FP16])
@pytest.mark.parametrize("model,integrator", [(gd.GD_ISING, gd.GD_EULER), (gd.GD_ISING, gd.GD_RK4),
                                              (gd.GD_XY, gd.GD_EULER), (gd.GD_XY, gd.GD_RK4)])
def test_same_bits_as_the_direct_to_lds_kernels(monkeypatch, prec, model, integrator):
    n, R = 512, 256
    rng = np.random.default_rng(21)
    vals = np.array([-448, -3, -1.5, -1, -0.015625, 0, 0.25, 1, 1.75, 6, 448], np.float32)
    J = I.sym_from_upper(rng.choice(vals, (n, n)).astype(np.float64))
    x = rng.uniform(-1, 1, (R, n) if model == gd.GD_ISING else (R, n, 2)).astype(np.float32)
    gam = rng.uniform(-0.5, 1.5, (R, n)).astype(np.float32)
    monkeypatch.setenv("GD_DENSE_CONFIG", "4")
    ref = _run(J, x, gam, prec, model, integrator)
    for cid in IDS:
        monkeypatch.setenv("GD_DENSE_CONFIG", str(cid))
        got = _run(J, x, gam, prec, model, integrator)
        for a, b in zip(ref[:3], got[:3]):
            assert np.array_equal(a, b), cid
        # device energies: FP32 coupling sums, their row tiles added in FP64
        assert np.abs(ref[3] - got[3]).max() <= 1e-12 * np.abs(ref[3]).max() + 1e-9, cid


@pytest.mark.parametrize("cid", IDS)
@pytest.mark.parametrize("n,R", [(33, 1), (200, 70), (700, 129), (1090, 257)])
def test_ragged_sizes_one_step_bound(monkeypatch, cid, n, R):
    monkeypatch.setenv("GD_DENSE_CONFIG", str(cid))
    J = I.sparse_pm1(n, 3)
    rng = np.random.default_rng(n)
    gam = rng.uniform(-0.5, 1.5, (R, n)).astype(np.float32)
    sub = sorted({0, R // 2, R - 1})
    _one_step_check(J, rng.uniform(-1.2, 1.2, (R, n)).astype(np.float32), gam, gd.GD_PREC_BF16, sub=sub)
    _one_step_check(J, rng.uniform(-1, 1, (R, n, 2)).astype(np.float32), gam, gd.GD_PREC_FP16, model="xy", sub=sub,
                    dt=0.02, integrator=gd.GD_RK4)
