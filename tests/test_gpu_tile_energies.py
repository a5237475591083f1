"""Device energies of the coupling kernels' energy mode, against integer energies
formed on the host from the same signs or states: the 32 x 32 tiles that compete
with the matrix-vector kernels, every tile on couplings in pieces (integers that
FP8 does not hold) and on complex amplitudes."""
import numpy as np
import pytest

from paper_1807_00699_amd import gd
from paper_1807_00699_amd import inputs as I

pytestmark = pytest.mark.gpu


def _energies(J, x, g):
    s = np.where(x < 0, -1, 1).astype(np.int64)
    J = J.astype(np.int64)
    return (-np.einsum("ri,ri->r", s, s @ J) + s @ g.astype(np.int64)).astype(np.float64)


@pytest.mark.parametrize("vals", [(-1, 0, 1), (-300, -1, 0, 7, 1000)])
@pytest.mark.parametrize("n,R,ids", [(200, 3, range(110, 126)), (200, 40, range(16)), (577, 16, range(110, 126))])
def test_integer_couplings(monkeypatch, n, R, ids, vals):
    rng = np.random.default_rng([n, R])
    J = I.sym_from_upper(rng.choice(np.array(vals, float), (n, n)))
    g = rng.integers(-3, 4, n).astype(np.float32)
    x = rng.uniform(-1, 1, (R, n)).astype(np.float32)
    want = _energies(J * (1 - np.eye(n, dtype=np.float32)), x, g)
    ran = 0
    for cid in ids:
        monkeypatch.setenv("GD_DENSE_CONFIG", str(cid))
        with gd.Solver(J, g) as S:
            try:
                S.set_state(x, np.zeros_like(x))
            except gd.GDError as e:
                assert e.code == gd.GD_E_INVALID_ARG and cid >= 110   # not a 32 x 32 tile
                continue
            E, b = S.energy(device_path=True)
            ran += 1
            assert np.array_equal(E, want) and b == int(np.argmin(want)), cid
    assert ran >= 2


@pytest.mark.parametrize("vals", [(-1, 0, 1), (-300, -1, 0, 7, 1000)])
def test_clock_states(monkeypatch, vals):
    """q = 4: states on the axes, integer energies."""
    n, R = 130, 9
    rng = np.random.default_rng(5)
    J = I.sym_from_upper(rng.choice(np.array(vals, float), (n, n)))
    k = rng.integers(0, 4, (R, n))
    th = np.pi / 2 * k + 0.3
    d0, d1 = np.array([1, 0, -1, 0])[k], np.array([0, 1, 0, -1])[k]
    Ji = (J * (1 - np.eye(n))).astype(np.int64)
    want = -(np.einsum("ri,ri->r", d0, d0 @ Ji) + np.einsum("ri,ri->r", d1, d1 @ Ji)).astype(np.float64)
    for cid in range(16):
        monkeypatch.setenv("GD_DENSE_CONFIG", str(cid))
        with gd.Solver(J, model=gd.GD_POTTS, q=4, h_q=0.1) as S:
            S.set_state(np.stack([np.cos(th), np.sin(th)], -1).astype(np.float32), np.zeros((R, n), np.float32))
            E, b = S.energy(device_path=True)
        assert np.array_equal(E, want) and b == int(np.argmin(want)), cid
