"""What setting up a state leaves behind: everything that asynchronous steps need
(they can be captured from the first call on), no form of J that nothing reads,
and no state at all when memory runs out."""
import ctypes

import numpy as np
import pytest

from paper_1807_00699_amd import gd
from paper_1807_00699_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,R,prec,coupling", [(200, 40, gd.GD_PREC_FP32, "pm1"), (200, 40, gd.GD_PREC_FP32, "gauss"),
                                               (64, 40, gd.GD_PREC_FP32, "pm1"), (200, 3, gd.GD_PREC_FP32, "gauss"),
                                               (200, 40, gd.GD_PREC_BF16, "pm1")])
def test_first_asynchronous_run_under_capture(n, R, prec, coupling):
    """Two captured runs of four steps (the state is back in its first buffers
    after them), replayed with eager work and synchronisation between, against
    eager ones."""
    import torch
    J = torch.from_numpy(I.dense_pm1(n, 3) if coupling == "pm1" else I.dense_gaussian(n, 3)).cuda()
    x0 = torch.from_numpy(I.psi0_real(n, R, 3)).cuda()
    st = torch.cuda.Stream()
    torch.cuda.synchronize()

    def make():
        p = gd.default_params(flags=gd.GD_F_DEVICE_PTRS | gd.GD_F_ASYNC, precision=prec, stream=st.cuda_stream)
        h = gd.gd_create(J, params=p)
        gd.gd_set_init(h, R, x0, device=True)
        return h

    def state(h):
        psi, gam = torch.empty((R, n), device="cuda"), torch.empty((R, n), device="cuda")
        torch.cuda.synchronize()
        assert gd.load().gd_get_state(h, ctypes.c_void_p(psi.data_ptr()), ctypes.c_void_p(gam.data_ptr()),
                                      None) == gd.GD_OK
        return psi.cpu().numpy(), gam.cpu().numpy()

    captured, eager = make(), make()
    try:
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            gd.gd_run(captured, R, 4)
            gd.gd_run(captured, R, 4)
        for _ in range(4):
            with torch.cuda.stream(st):
                g.replay()
            gd.gd_run(eager, R, 4)
            gd.gd_run(eager, R, 4)
            torch.cuda.synchronize()
            for a, b in zip(state(captured), state(eager)):
                assert np.array_equal(a, b)
    finally:
        gd.gd_destroy(captured)
        gd.gd_destroy(eager)


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_no_second_copy_of_j_for_matrix_vector_steps(monkeypatch):
    """N = 4096, couplings that are not exact in FP8: 64 MiB of J; its pieces for
    the coupling kernels would be 96 MiB more."""
    n, R = 4096, 8
    J, x0 = I.dense_gaussian(n, 2), I.psi0_real(n, R, 2)
    monkeypatch.setenv("GD_DENSE_CONFIG", "101")
    with gd.Solver(I.dense_gaussian(64, 2)) as S:    # (the library's own set-up)
        S.set_init(1)
        S.run(1)
    before = _free()
    with gd.Solver(J) as S:
        S.set_init(R, x0)
        S.run(2)
        S.energy(device_path=True)
        assert S.stats().kernel_config == 101
        used = before - _free()
    assert 64 << 20 <= used <= (64 + 48) << 20


def test_no_state_without_memory_for_it():
    """The coupling kernels' form of J (1.5 GiB) does not fit: an error and no
    state; once there is room the same solver works."""
    import torch
    n, R = 16384, 128
    J = np.zeros((n, n), np.float32)
    J[0, 1:] = J[1:, 0] = np.linspace(0.1, 1.0, n - 1, dtype=np.float32)
    with gd.Solver(J) as S:
        keep = [torch.empty(max(_free() - (2 << 30), 1), dtype=torch.uint8, device="cuda")]
        try:        # (more may be free than is reported)
            while True:
                keep.append(torch.empty(128 << 20, dtype=torch.uint8, device="cuda"))
        except torch.cuda.OutOfMemoryError:
            pass
        del keep[-8:]
        torch.cuda.empty_cache()    # 1 GiB and less than 128 MiB more
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
