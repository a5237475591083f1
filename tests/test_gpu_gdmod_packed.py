"""GD-mod with one triangle of every K (sets of K past the last-level cache):
ragged sizes around the 64-wide tiles, real and complex, against the oracle
with test_gpu_gdmod's bar, and K read back whole."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1807_00699_amd import gd
from paper_1807_00699_amd import inputs as I
from test_gpu_gdmod import TOL, _gamma_c, _rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,n,R", [("ising", 65, 1600), ("ising", 577, 62), ("xy", 640, 62), ("xy", 130, 700)])
def test_packed_couplings_parity(model, n, R):
    assert R * (-(-n // 64) * 64) ** 2 >= 25_000_000
    J = I.dense_gaussian(n, 4)
    psi0 = I.psi0_complex(n, R, 4) if model == "xy" else I.psi0_real(n, R, 4)
    gc = _gamma_c(J)
    sub = [0, R // 2, R - 1]
    with gd.Solver(J, model=gd.GD_XY if model == "xy" else gd.GD_ISING, dt=0.02, eps=0.1,
                   variant=gd.GD_VARIANT_MOD, eps_hat=0.2, gamma_c=gc) as S:
        S.set_init(R, psi0)
        assert np.array_equal(S.mod_couplings(R - 1), J * (1 - np.eye(n, dtype=np.float32)))
        S.run(60)
        p, gm, _ = S.state()
        Kg = np.stack([S.mod_couplings(r) for r in sub])
        s = S.scale
    assert np.array_equal(Kg, Kg.transpose(0, 2, 1))
    op, og, oK = O.run_mod(J, psi0[sub], model=model, steps=60, dt=0.02, eps=0.1, eps_hat=0.2, gamma_c=gc, s=s)
    assert _rel(p[sub], op).max() <= TOL and _rel(gm[sub], og).max() <= TOL
    assert _rel(Kg, oK).max() <= TOL


@pytest.mark.parametrize("model,n,R", [("xy", 200, 16), ("ising", 200, 16), ("xy", 640, 62)])
def test_checks_during_a_run(model, n, R):
    """Energy checks of a GD-mod run (the coupling kernels' form of J is laid out
    for them): the last one's best is that of the energies of the same state."""
    J = I.dense_pm1(n, 7)
    psi0 = I.psi0_complex(n, R, 7) if model == "xy" else I.psi0_real(n, R, 7)
    with gd.Solver(J, model=gd.GD_XY if model == "xy" else gd.GD_ISING, dt=0.02, eps=0.1, variant=gd.GD_VARIANT_MOD,
                   eps_hat=0.2, gamma_c=_gamma_c(J), check_interval=12) as S:
        S.set_init(R, psi0)
        S.run(12)
        st = S.stats()
        Ed, _ = S.energy(device_path=True)
    assert st.best_index == int(np.argmin(Ed)) and st.best_energy == Ed.min()
