"""The one-pass bin sort: the edges of its rule, its batches and its bins."""
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


# 1024 bins (m = 31, a grid of 256 cells per axis), 16 (m = 7), 4 (m = 3), and 4096 (m = 32, two passes); 4095
# points (two passes) and 4096; one point more than a batch of 8192 and of 4096; all points in one bin or one row
@pytest.mark.parametrize("m,n,ntgt,dtype,shape", [
    (31, 4095, 1, "float32", "flat"), (31, 4096, 1, "float32", "flat"), (31, 8193, 0, "float32", "flat"),
    (31, 8193, 1, "float32", "flat"), (31, 4097, 2, "float64", "flat"), (31, 20_011, 3, "float32", "row"),
    (31, 20_011, 7, "float64", "bin"), (31, 20_011, 0, "float64", "bin"), (32, 20_011, 1, "float32", "row"),
    (7, 30_011, 5, "float32", "flat"), (3, 30_011, 1, "float64", "row"), (3, 30_011, 4, "float32", "bin")])
def test_one_pass_edges(fk, m, n, ntgt, dtype, shape):
    import torch
    rng = np.random.default_rng(n + ntgt + m)
    X = rng.uniform(-np.pi, np.pi, (2, n))
    if shape != "flat":
        X[0, : n - 5] = 0.3 + 1e-3 * X[0, : n - 5]
    if shape == "bin":
        X[1, : n - 5] = -2.0 + 1e-3 * X[1, : n - 5]
    X = X.astype(dtype)
    Y = rng.standard_normal((max(ntgt, 1), n)).astype(dtype)
    M, b = fk.gram(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda() if ntgt else None, m)
    X, Y = X.astype(np.float64), Y.astype(np.float64)
    # the type-1 bars: 1e-6 of M[0] for M, 1e-6 of the mean |Y| for b (targets are rounded to FP32: 6e-8)
    assert np.abs(M.cpu().numpy() - oracle.gram_generator(X, m)).max() <= 1e-6
    if ntgt:
        err = np.abs(b.cpu().numpy() - oracle.rhs(X, Y, m)).max(axis=1)
        assert (err <= 1.1e-6 * np.abs(Y).mean(axis=1)).all()
