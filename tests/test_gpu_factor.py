"""The FP32 factorization's diagonal-block kernels at the edges of their blocks and of their dispatch."""
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


# N = 2m + 1 unknowns in blocks of 64: one partly filled block, one block less and plus one row, two and
# three blocks; 350 lambdas x 3 block rows exceed the workgroups that solve a panel with its diagonal
# block, 340 do not.
@pytest.mark.parametrize("m,nlam", [(1, 1), (31, 2), (32, 1), (63, 3), (64, 1), (64, 340), (64, 350)])
def test_factor_block_edges(fk, m, nlam):
    import torch
    rng = np.random.default_rng(m * 1000 + nlam)
    n = 400
    X = rng.uniform(-np.pi, np.pi, (1, n))
    X = X + 0.5 * np.sin(X)
    Y = rng.standard_normal((2, n))
    M, b = oracle.gram_generator(X, m), oracle.rhs(X, Y, m)
    lams = list(10.0 ** np.linspace(-4, -1, nlam))
    p = oracle.sobolev_weights(m, 1, 1.0)
    # tolerance: the refined residual is at most 1e-10 ||b||, so the error is at most kappa times that
    th, info = fk.solve(torch.from_numpy(M).cuda(), torch.from_numpy(b).cuda(), m, lams, penalty="sobolev", s=1.0,
                        info=True)
    assert info["refine_iters"] <= 2          # an FP32-class factor at these condition numbers (< 1e5)
    th = th.cpu().numpy()
    for i in sorted({0, nlam // 2, nlam - 1}):
        A = oracle.system_matrix(M, m, lams[i], p)
        want = oracle.solve_system(A, b)
        kappa = np.linalg.cond(A)
        for t in range(2):
            err = np.linalg.norm(th[i, t] - want[t]) / np.linalg.norm(want[t])
            assert err <= 1e-10 * kappa + 1e-13, (i, t, err, kappa)


@pytest.mark.parametrize("m,nlam", [(10, 1), (64, 1), (64, 350)])
def test_non_positive_pivot_is_reported(fk, m, nlam):
    """-1 on the Gram's diagonal: the first pivot is negative in every block kernel."""
    import torch
    M = np.zeros(4 * m + 1, dtype=np.complex128)
    M[2 * m] = -1.0
    b = np.ones((1, 2 * m + 1), dtype=np.complex128)
    with pytest.raises(fk.FkError) as e:
        fk.solve(torch.from_numpy(M).cuda(), torch.from_numpy(b).cuda(), m, [1e-3] * nlam, penalty="identity")
    assert e.value.code == 4
