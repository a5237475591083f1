"""Persistent steps of few trajectories on couplings that are exact in FP8: the
one-byte copy of J and FP32 J (GD_J8_COPY=0) give the same bits."""
import numpy as np
import pytest

from paper_1807_00699_amd import gd
from paper_1807_00699_amd import inputs as I
from test_gpu_persist import K, _solver, _start

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,R", [(129, 1), (577, 3), (1000, 4), (2048, 2), (4096, 1), (4096, 4)])
def test_copy_of_j_or_not(monkeypatch, n, R):
    rng = np.random.default_rng(n)
    J = I.sym_from_upper(rng.choice(np.array([-448, -3, -1.5, -0.015625, 0, 0.25, 1, 6, 44.0]), (n, n)))
    x0, g0 = _start("ising", n, R)
    out = []
    for copy in ("1", "0"):
        monkeypatch.setenv("GD_J8_COPY", copy)
        with _solver(J, "ising", False) as S:
            S.set_state(x0, g0)
            S.run(K)
            assert S.stats().kernel_config >= 208
            out.append(S.state()[:2])
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
