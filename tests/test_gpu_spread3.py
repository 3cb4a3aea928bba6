"""The 3-D sort and spread: kernel widths, channel groups, batches and slices of a bin."""
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


# eps: kernel widths below 7, 7 and 8 (patches of one cell); T + 1 channels in groups
# of 1 .. 4; "one": nearly all points in one bin (several slices, batches of 256)
@pytest.mark.parametrize("m,T,n,eps,shape", [(4, 0, 5_000, 1e-3, "flat"), (4, 1, 40_001, 2e-7, "flat"),
                                             (4, 2, 20_000, 2e-7, "one"), (3, 3, 9_000, 2e-7, "flat"),
                                             (3, 4, 30_001, 2e-7, "one"), (7, 8, 6_001, 2e-7, "flat"),
                                             (5, 5, 257, 2e-7, "flat"),
                                             (1, 1, 1, 2e-7, "flat"), (8, 1, 70_000, 2e-7, "flat")])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_gram_3d(fk, m, T, n, eps, shape, dtype):
    import torch
    rng = np.random.default_rng(17 * m + n)
    X = rng.uniform(-np.pi, np.pi, (3, n))
    if shape == "one":
        X[:, 3:] = 0.4 + 1e-2 * X[:, 3:]
    X = X.astype(dtype)
    Y = rng.standard_normal((max(T, 1), n)).astype(dtype)
    ctx = fk.Context(0, eps=eps)
    M, b, info = fk.gram(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda() if T else None, m, ctx=ctx, info=True)
    assert info["bin"] == 8
    X64, Y64 = X.astype(np.float64), Y.astype(np.float64)
    # three axes of kernel error eps, FP32 products (6e-8 each, three factors), targets rounded to FP32
    tol = 4 * eps + 4e-7
    assert np.abs(M.cpu().numpy() - oracle.gram_generator(X64, m)).max() <= tol
    if T:
        err = np.abs(b.cpu().numpy() - oracle.rhs(X64, Y64, m)).max(axis=1)
        assert (err <= tol * np.abs(Y64).mean(axis=1)).all()


def test_gram_3d_reports_bad_input(fk):
    import torch
    X = torch.zeros((3, 100), device="cuda")
    Y = torch.zeros((2, 100), device="cuda")
    Y[1, 7] = float("nan")
    with pytest.raises(fk.FkError) as e:
        fk.gram(X, Y, 4)
    assert e.value.code == 3
    X[2, 9] = 7.0
    with pytest.raises(fk.FkError) as e:
        fk.gram(X, None, 4)
    assert e.value.code == 2
