"""FP32 coupling kernels on the BF16 matrix cores (gd_split.h): every variant at
the edges of its tiles.  Sizes around one and two 64-wide row paddings, row
tiles that end past the matrix, one trajectory, and trajectory counts that
leave partial column tiles; FP8-stored and split couplings, real and complex.

One Euler step from a given state against float64, within the rounding
envelope of an FP32 evaluation: |x1 - x1'| <= 2 (n + 8) 2^-24 (|x1| + dt M),
M = |x| (|gamma| + |x|^2) + sum_j |J_ij| |x_j| / s.  Integer couplings: the
device energies equal the FP64 re-score exactly."""
import numpy as np
import pytest

from paper_1807_00699_amd import gd
from paper_1807_00699_amd import inputs as I

pytestmark = pytest.mark.gpu

VARIANTS = range(16)
DT = 0.05


@pytest.mark.parametrize("coupling", ["pm1", "uniform"])
@pytest.mark.parametrize("model", ["ising", "xy"])
@pytest.mark.parametrize("n,R", [(33, 1), (65, 130), (200, 31), (320, 70)])
def test_every_variant_one_step_at_tile_edges(monkeypatch, n, R, model, coupling):
    J = I.dense_pm1(n, 3) if coupling == "pm1" else I.dense_uniform(n, 3)
    cx = model == "xy"
    # amplitudes over four decades: every piece of the split carries weight
    rng = np.random.default_rng([n, R])
    mag = 10.0 ** rng.uniform(-4, 0, (R, n, 2 if cx else 1))
    psi = (mag * rng.choice([-1.0, 1.0], mag.shape)).astype(np.float32)
    gam = rng.uniform(-1, 1, (R, n)).astype(np.float32)
    J64, p64, g64 = J.astype(np.float64), psi.astype(np.float64), gam.astype(np.float64)
    s = np.sqrt((J64 ** 2).sum() / n)
    rho = (p64 ** 2).sum(-1)
    C = np.einsum("ij,rjp->rip", J64, p64) / s
    want = p64 + DT * (p64 * (g64 - rho)[..., None] + C)
    M = np.abs(p64) * (np.abs(g64) + rho)[..., None] + np.einsum("ij,rjp->rip", np.abs(J64), np.abs(p64)) / s
    bound = 2 * (n + 8) * 2.0**-24 * (np.abs(want) + DT * M)
    gwant = g64 + DT * 0.1 * (1.0 - rho)
    gbound = 2 * 8 * 2.0**-24 * (np.abs(gwant) + DT * (1.0 + rho))
    for cid in VARIANTS:
        monkeypatch.setenv("GD_DENSE_CONFIG", str(cid))
        with gd.Solver(J, model=gd.GD_XY if cx else gd.GD_ISING, dt=DT, eps=0.1) as S:
            S.set_state(psi if cx else psi[..., 0], gam)
            S.run(1)
            x, g, _ = S.state()
            E, _ = S.energy()
            Ed, _ = S.energy(device_path=True)
        x = x.reshape(R, n, -1)
        assert np.all(np.abs(x - want) <= bound), (cid, np.max(np.abs(x - want) / bound))
        assert np.all(np.abs(g - gwant) <= gbound), cid
        if coupling == "pm1" and not cx:
            assert np.array_equal(E, Ed), cid
        else:
            assert np.allclose(E, Ed, rtol=0, atol=2e-5 * np.abs(J64).sum() / n**0.5), cid


@pytest.mark.parametrize("model,prec", [(gd.GD_ISING, gd.GD_PREC_FP32), (gd.GD_ISING, gd.GD_PREC_BF16),
                                        (gd.GD_ISING_COMPLEX, gd.GD_PREC_FP32)])
@pytest.mark.parametrize("n,R", [(2, 1), (33, 5), (65, 130), (320, 31), (1100, 1200)])
def test_sign_energies_exact(n, R, model, prec):
    """Energies from the signs of the amplitudes (FP8-stored couplings), at the
    edges of the tiles: exactly sum_i -s_i (J s)_i + g_i s_i in integers for
    integer couplings (up to 448 in magnitude) and fields, +0, -0 and
    subnormal amplitudes reading as +1, -1 where negative; couplings in halves
    take the FP64 re-score: 1e-12 of sum |J| there."""
    rng = np.random.default_rng([n, R, 9])
    s = np.where(rng.random((R, n)) < 0.5, -1.0, 1.0)
    amp = (s * rng.choice([1.0, 0.25, 1e-30, 1e-41], (R, n))).astype(np.float32)
    zero = rng.random((R, n)) < 0.1
    amp[zero] = np.where(s[zero] < 0, -0.0, 0.0)
    s = np.where(amp < 0, -1.0, 1.0)
    psi = amp if model == gd.GD_ISING else np.stack([amp, rng.uniform(-1, 1, amp.shape).astype(np.float32)], -1)
    for half in (False, True):
        vals = np.array([-448, -208, -9, -3, -1, 0, 1, 2, 10, 44]) if not half else np.array([-1.5, -1.0, 0.0, 0.5, 2.0])
        J = I.sym_from_upper(rng.choice(vals, (n, n)))
        g = rng.integers(-3, 4, n).astype(np.float32)
        J64 = J.astype(np.float64)
        want = -np.einsum("ri,ri->r", s, s @ J64) + s @ g.astype(np.float64)
        with gd.Solver(J, g, model=model, precision=prec) as S:
            S.set_state(psi, np.zeros((R, n), np.float32))
            E, b = S.energy()
            Ed, bd = S.energy(device_path=True)
        tol = 1e-12 * np.abs(J64).sum()
        assert np.all(np.abs(E - want) <= (tol if half else 0.0))
        if not half:
            assert np.array_equal(Ed, want) and b == bd == int(np.argmin(want))
