"""gd_mod_couplings of packed and full K with GD_F_DEVICE_PTRS: into device memory
(whole words in the middle of an allocation, an unaligned address), into pinned
host memory; pageable host memory is refused with an error code, which no later
call reports again.  Nothing but an allocation of the solver's device may be
written by a kernel."""
import ctypes

import numpy as np
import pytest

from paper_1807_00699_amd import gd
from paper_1807_00699_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,R", [(130, 4), (130, 700), (577, 62)])
def test_destinations(n, R):
    import torch
    lib = gd.load()
    J = I.dense_gaussian(n, 4)
    want = J * (1 - np.eye(n, dtype=np.float32))
    Jd = torch.from_numpy(J).cuda()
    torch.cuda.synchronize()
    h = gd.gd_create(Jd, model=gd.GD_ISING, params=gd.default_params(variant=gd.GD_VARIANT_MOD, gamma_c=50.0,
                                                                     flags=gd.GD_F_DEVICE_PTRS))
    try:
        gd.gd_set_init(h, R)
        for off in (0, 4, 12, 1, 2):
            t = torch.full((4 * n * n + 64,), 7, dtype=torch.uint8, device="cuda")
            torch.cuda.synchronize()
            assert lib.gd_mod_couplings(h, R - 1, ctypes.c_void_p(t.data_ptr() + off)) == gd.GD_OK, off
            b = t.cpu().numpy()
            assert b[off:off + 4 * n * n].tobytes() == want.tobytes()
            assert np.all(b[:off] == 7) and np.all(b[off + 4 * n * n:] == 7)
        pinned = torch.zeros((n, n), pin_memory=True)
        assert lib.gd_mod_couplings(h, 0, ctypes.c_void_p(pinned.data_ptr())) == gd.GD_OK
        assert np.array_equal(pinned.numpy(), want)
        paged = np.zeros((n, n), np.float32)
        assert lib.gd_mod_couplings(h, 0, paged.ctypes.data_as(ctypes.c_void_p)) == gd.GD_E_DEVICE
        gd.gd_set_init(h, R)    # the error is reported once
    finally:
        gd.gd_destroy(h)
