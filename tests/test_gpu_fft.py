"""The type-1 stage's transforms at every grid length, with odd and even numbers of lines."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fk():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2509_02649_amd as fk
    return fk


# grids of 16 (m = 1) to 1024 (m = 64) points per axis; C = T + 1 lines (1-D) odd and even
@pytest.mark.parametrize("d,m,T", [(1, 1, 1), (1, 3, 2), (1, 7, 1), (1, 15, 0), (1, 31, 3), (1, 63, 2), (1, 64, 1),
                                   (2, 1, 0), (2, 3, 1), (2, 7, 2), (2, 31, 1), (2, 63, 0), (2, 64, 1),
                                   (3, 1, 1), (3, 3, 0), (3, 7, 2), (3, 15, 1)])
def test_every_grid_length(fk, d, m, T):
    import torch
    rng = np.random.default_rng(100 * d + m)
    n = 3001
    X = rng.uniform(-np.pi, np.pi, (d, n))
    Y = rng.standard_normal((max(T, 1), n))
    M, b = fk.gram(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda() if T else None, m)
    # the type-1 bars: 1e-6 of M[0], 1e-6 of the mean |Y| (targets rounded to FP32: 6e-8)
    assert np.abs(M.cpu().numpy() - oracle.gram_generator(X, m)).max() <= 1e-6
    if T:
        err = np.abs(b.cpu().numpy() - oracle.rhs(X, Y, m)).max(axis=1)
        assert (err <= 1.1e-6 * np.abs(Y).mean(axis=1)).all()
