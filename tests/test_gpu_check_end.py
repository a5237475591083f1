"""The end of energy checks and runs on both sides of the trajectory counts where
it moves between the last workgroup of the kernel before it and a launch of its
own: best energy and trajectory, the energy trace, and the trajectories that
diverged."""
import numpy as np
import pytest

from paper_1807_00699_amd import gd
from paper_1807_00699_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,R", [(20, 1), (20, 256), (20, 257), (100, 4097), (64, 20000), (300, 256), (300, 257),
                                 (300, 512), (300, 513)])
def test_best_trace_and_diverged(n, R):
    J = I.dense_pm1(n, 3)
    x0 = I.psi0_real(n, R, 3)
    with gd.Solver(J, check_interval=6) as S:
        S.set_init(R, x0)
        S.run(18)
        st = S.stats()
        E, b = S.energy()
        steps, trace = gd.gd_best_trace(S.h)
        assert list(steps) == [6, 12, 18] and st.best_energy == trace[-1] <= E.min()
        if trace[-1] < trace[-2]:
            assert st.best_index == b == int(np.argmin(E)) and trace[-1] == E.min()
        x, g, _ = S.state()
        bad = sorted({0, R // 2, R - 1})
        x[bad, 0] = 1e30           # cubed past the largest float
        S.set_state(x, g)
        with pytest.raises(gd.GDError) as e:
            S.run(6)
        assert e.value.code == gd.GD_E_DIVERGED and S.stats().diverged == len(bad)
        assert list(np.flatnonzero(S.trajectory_status())) == bad
