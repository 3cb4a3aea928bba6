"""The 1-D spread with copies of its grid in LDS: the edge of its rule and each number of copies."""
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


# grids of 512 cells (m = 64) hold 32, 16, 8, 4, 2 and 1 copies with 0, 1, 3, 8, 17 and 32 targets, smaller ones more
@pytest.mark.parametrize("n,m,ntgt,dtype", [(2 ** 19 - 1, 64, 1, "float32"), (2 ** 19, 64, 0, "float32"),
                                            (2 ** 19, 64, 1, "float64"), (2 ** 19 + 1, 64, 3, "float32"),
                                            (2 ** 19 + 1, 60, 8, "float32"), (2 ** 19 + 1, 64, 17, "float32"),
                                            (2 ** 19 + 1, 64, 32, "float32"), (600_001, 3, 2, "float64")])
def test_copies(fk, n, m, ntgt, dtype):
    import torch
    rng = np.random.default_rng(m + ntgt)
    X = rng.uniform(-np.pi, np.pi, (1, n))
    X[0, : n // 3] = 0.3 + 1e-4 * X[0, : n // 3]    # many points in one cell
    X = X.astype(dtype)
    Y = rng.standard_normal((max(ntgt, 1), n)).astype(dtype)
    M, b = fk.gram(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda() if ntgt else None, m)
    X, Y = X.astype(np.float64), Y.astype(np.float64)
    # the type-1 bars: 1e-6 of M[0] for M, 1e-6 of the mean |Y| for b (targets are rounded to FP32: 6e-8)
    assert np.abs(M.cpu().numpy() - oracle.gram_generator(X, m)).max() <= 1e-6
    if ntgt:
        err = np.abs(b.cpu().numpy() - oracle.rhs(X, Y, m)).max(axis=1)
        assert (err <= 1.1e-6 * np.abs(Y).mean(axis=1)).all()
