"""FP16 inference reads a packed copy of the parameters: it follows every change
of them (training steps, assignment), bit for bit the outputs of a new network
with the same parameters; rows around the tile of 32 and the grid's stride."""
import numpy as np
import pytest

from paper_1807_00699_amd import gd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 31, 33, 65537, 200003])
def test_inference_follows_the_parameters(M):
    rng = np.random.default_rng(M)
    X = rng.normal(size=(M, gd.GD_NFEAT)).astype(np.float32)
    lab = np.where(rng.random(M) < 0.5, -1.0, 1.0).astype(np.float32)
    seg = np.array([0, M], np.int32)
    with gd.MLP(seed=3) as m:
        for step in range(3):
            got = m.forward(X, fp16=True)
            with gd.MLP(params=m.params) as fresh:
                assert np.array_equal(got, fresh.forward(X, fp16=True)), step
            ref = m.forward(X)                      # FP32, from the parameters themselves
            assert np.abs(got - ref).max() <= 0.05 * max(1.0, np.abs(ref).max()), step
            if step == 0:
                m.train_step(X, lab, seg, 1e-2)
            else:
                m.params = (0.5 * rng.normal(size=gd.GD_MLP_NPARAM) / 8).astype(np.float32)
