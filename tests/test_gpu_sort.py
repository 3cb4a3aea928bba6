"""The two-pass bin sort at the edges of its workgroups and slices."""
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


# First-pass workgroups take at least 8192 points; second-pass slices at least 4096, and a row that holds
# nearly all points has many of them while the others have one or none.
@pytest.mark.parametrize("ntgt", [0, 1, 3, 16])
@pytest.mark.parametrize("n,shape", [(8191, "flat"), (8193, "flat"), (16385, "flat"), (150_001, "row"),
                                     (150_001, "column")])
def test_sort_edges(fk, ntgt, n, shape):
    import torch
    rng = np.random.default_rng(n + ntgt)
    X = rng.uniform(-np.pi, np.pi, (2, n))
    if shape != "flat":
        a = 0 if shape == "row" else 1
        X[a, : n - 5] = 0.3 + 1e-3 * X[a, : n - 5]
    Y = rng.standard_normal((max(ntgt, 1), n))
    m = 6
    M, b = fk.gram(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda() if ntgt else None, m)
    # the type-1 bars: 1e-6 of M[0] for M, 1e-6 of the mean |Y| for b (targets are rounded to FP32: 6e-8)
    assert np.abs(M.cpu().numpy() - oracle.gram_generator(X, m)).max() <= 1e-6
    if ntgt:
        err = np.abs(b.cpu().numpy() - oracle.rhs(X, Y, m)).max(axis=1)
        assert (err <= 1.1e-6 * np.abs(Y).mean(axis=1)).all()
