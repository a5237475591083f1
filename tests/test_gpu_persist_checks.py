"""Steps between energy checks: persistent from four coupling evaluations between
two checks on, one launch per step below; the same trajectory and the energies
of the checked states on both sides of that line.

Tolerance: two evaluations of test_gpu_persist's steps."""
import numpy as np
import pytest

from paper_1807_00699_amd import gd
from paper_1807_00699_amd import inputs as I
from test_gpu_persist import DT, K, TOL, _start

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,n,R,rk4", [("ising", 700, 2, False), ("ising", 300, 20, False), ("xy", 300, 9, False),
                                           ("xy", 300, 9, True)])
def test_check_intervals_around_the_line(model, n, R, rk4):
    J = I.sparse_pm1(n, 6)
    x0, g0 = _start(model, n, R)
    out = []
    for check in (0, 1, 2, 3, 4, 5):
        with gd.Solver(J, model=gd.GD_ISING if model == "ising" else gd.GD_XY, dt=DT, eps=0.1, check_interval=check,
                       integrator=gd.GD_RK4 if rk4 else gd.GD_EULER) as S:
            S.set_state(x0, g0)
            S.run(K)
            st = S.stats()
            assert (st.kernel_config >= 200) == (check == 0 or check * (4 if rk4 else 1) >= 4)
            out.append(S.state()[:2])
            if check == 1:
                E, b = S.energy(device_path=True)
                steps, trace = S.best_trace()
                assert list(steps) == list(range(1, K + 1)) and trace[-1] == st.best_energy <= E.min()
    for x, g in out[1:]:
        assert np.linalg.norm(x - out[0][0]) <= 2 * TOL * np.linalg.norm(out[0][0])
        assert np.linalg.norm(g - out[0][1]) <= 2 * TOL * np.linalg.norm(out[0][1])
