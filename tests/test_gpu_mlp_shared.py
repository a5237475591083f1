"""One network used by several threads and streams right after its parameters
changed: every proposal is that of the new parameters."""
import threading

import numpy as np
import pytest

from paper_1807_00699_amd import gd
from paper_1807_00699_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_proposals_of_several_threads_follow_the_parameters():
    rng = np.random.default_rng(4)
    R, total = 4, 20 + 33 + 64
    inst = [dict(n=n, J=I.dense_pm1(n, n)) for n in (20, 33, 64)]
    solvers = [gd.BatchSolver(inst) for _ in range(6)]
    X = rng.normal(size=(900, gd.GD_NFEAT)).astype(np.float32)
    lab = np.where(rng.random(900) < 0.5, -1.0, 1.0).astype(np.float32)
    seg = np.array([0, 400, 900], np.int32)
    try:
        with gd.MLP(seed=1) as m:
            for rep in range(24):
                if rep % 2:
                    m.params = (rng.normal(size=gd.GD_MLP_NPARAM) / 8).astype(np.float32)
                else:
                    m.train_step(X, lab, seg, 0.05)
                with gd.MLP(params=m.params) as fresh:
                    gd.gd_propose(solvers[0].h, fresh, R, 5, 0.5, 0.1, 9)
                    want = gd.gd_get_state(solvers[0].h, R, total, False)[0]
                go = threading.Barrier(len(solvers))

                def work(S):
                    go.wait()
                    gd.gd_propose(S.h, m, R, 5, 0.5, 0.1, 9)

                th = [threading.Thread(target=work, args=(S,)) for S in solvers]
                for t in th:
                    t.start()
                for t in th:
                    t.join()
                for S in solvers:
                    assert np.array_equal(gd.gd_get_state(S.h, R, total, False)[0], want), rep
    finally:
        for S in solvers:
            S.close()
