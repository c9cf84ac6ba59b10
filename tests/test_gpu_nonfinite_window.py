"""A loaded window that is not finite has rank 0, whatever the solve's size class:
no singular value of it is reported as one."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [6, 20, 50, 90, 120, 180, 250])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_rank_zero(m, bad):
    import paper_1612_07875_amd as dmd
    n = 300
    rng = np.random.default_rng(m)
    X = rng.standard_normal((m + 1, n))
    for r in (1, 5):
        for column in (0, 1, m // 2, m - 1):
            Y = X.copy()
            Y[column, 77] = bad
            with dmd.Stream(n, m, r, dtype="f64") as s:
                s.load_window(torch.from_numpy(Y).cuda())
                s.solve()
                sigma, V, status = s.svd()
                assert status > 0 and V.shape == (m, 0) and (sigma == 0).all(), (r, column, status)
                lam, _, status = s.eigs()
                assert status > 0 and lam.size == 0
                s.load_window(torch.from_numpy(X).cuda())  # and the handle goes on
                s.solve()
                sigma, V, status = s.svd()
                ref = np.sqrt(np.linalg.eigvalsh(X[:m] @ X[:m].T)[::-1])
                assert status == 0 and np.allclose(sigma, ref, rtol=1e-9)
