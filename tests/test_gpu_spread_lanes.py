"""The 2-D spread of 17 and more channels with lanes over the channels: odd points, one or two points at a time."""
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


# 31 targets and fewer: two points at a time, 32: one; batches of 64 points with 1, 7, 63 and 64 in the last; all points
# in one bin (many batches, several waves) or spread over all bins
@pytest.mark.parametrize("ntgt,n,m,dtype,shape", [(17, 65, 8, "float32", "bin"),
                                                  (20, 4097, 32, "float32", "flat"), (31, 20_011, 20, "float64", "bin"),
                                                  (31, 1087, 8, "float32", "bin"), (32, 1088, 8, "float32", "bin"),
                                                  (32, 20_011, 32, "float64", "flat"), (32, 7, 16, "float32", "bin")])
def test_many_channels(fk, ntgt, n, m, dtype, shape):
    import torch
    rng = np.random.default_rng(n + ntgt)
    X = rng.uniform(-np.pi, np.pi, (2, n))
    if shape == "bin":
        X = 0.3 + 1e-3 * X
    X = X.astype(dtype)
    Y = rng.standard_normal((ntgt, n)).astype(dtype)
    M, b = fk.gram(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), m)
    X, Y = X.astype(np.float64), Y.astype(np.float64)
    # the type-1 bars: 1e-6 of M[0] for M, 1e-6 of the mean |Y| for b (targets are rounded to FP32: 6e-8)
    assert np.abs(M.cpu().numpy() - oracle.gram_generator(X, m)).max() <= 1e-6
    err = np.abs(b.cpu().numpy() - oracle.rhs(X, Y, m)).max(axis=1)
    assert (err <= 1.1e-6 * np.abs(Y).mean(axis=1)).all()
