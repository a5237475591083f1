"""Setting up a state leaves none behind when memory runs out."""
import numpy as np
import pytest

from paper_1807_00699_amd import gd
from paper_1807_00699_amd import inputs as I

pytestmark = pytest.mark.gpu


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_no_state_without_memory_for_it():
    """The coupling kernels' form of J (1.5 GiB) does not fit: an error and no
    state; once there is room the same solver works."""
    import torch
    n, R = 16384, 128
    J = np.zeros((n, n), np.float32)
    J[0, 1:] = J[1:, 0] = np.linspace(0.1, 1.0, n - 1, dtype=np.float32)
    with gd.Solver(J) as S:
        keep = torch.empty(_free() - (1 << 30), dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        with pytest.raises(gd.GDError) as e:
            S.set_init(R)
        assert e.value.code == gd.GD_E_OOM
        with pytest.raises(gd.GDError) as e:
            gd.gd_energy(S.h, R)
        assert e.value.code == gd.GD_E_STATE
        del keep
        torch.cuda.empty_cache()
        S.set_init(R)
        S.run(1)
        assert np.all(np.isfinite(S.state()[0]))
