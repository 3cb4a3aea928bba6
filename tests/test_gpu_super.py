"""Solves through inverted super-blocks, and the residual by rows: edges of blocks and of the dispatch."""
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


# N = (2m + 1)^d unknowns, nb = ceil(N / 64) block columns: 3 (the fewest), 4 and 5, 8 and 9 (one super-block
# and one more block), 15, 27; 1 and 2 column tiles (targets), 1 .. 5 column tiles of the residual; 100 x 10
# block columns x lambdas within the rule, 100 x 12 past it
@pytest.mark.parametrize("d,m,nlam,T", [(1, 64, 1, 1), (2, 7, 2, 16), (2, 8, 1, 17), (2, 10, 3, 2), (2, 11, 1, 32),
                                        (2, 15, 5, 5), (2, 20, 2, 1), (2, 12, 100, 1), (2, 13, 100, 1)])
def test_super_block_solves(fk, d, m, nlam, T):
    import torch
    rng = np.random.default_rng(1000 * m + nlam)
    X = rng.uniform(-np.pi, np.pi, (d, 3000))
    X = X + 0.5 * np.sin(X)
    Y = rng.standard_normal((T, 3000))
    M, b = oracle.gram_generator(X, m), oracle.rhs(X, Y, m)
    lams = list(10.0 ** np.linspace(-4, -1, nlam))
    p = oracle.sobolev_weights(m, d, 1.0)
    ctx = fk.Context(0)
    th, info = fk.solve(torch.from_numpy(M).cuda(), torch.from_numpy(b).cuda(), m, lams, penalty="sobolev", s=1.0,
                        ctx=ctx, info=True)
    assert info["refine_iters"] <= 2
    th = th.cpu().numpy()
    # one unrefined solve: FP32-class, kappa(A) 2^-24 with a factor for the sums over N terms
    ctx0 = fk.Context(0, max_refine=0, refine_tol=1e-2)
    th0 = fk.solve(torch.from_numpy(M).cuda(), torch.from_numpy(b).cuda(), m, lams, penalty="sobolev", s=1.0,
                   ctx=ctx0).cpu().numpy()
    for i in sorted({0, nlam - 1}):
        A = oracle.system_matrix(M, m, lams[i], p)
        want = oracle.solve_system(A, b)
        kappa = np.linalg.cond(A)
        for t in range(T):
            n = np.linalg.norm(want[t])
            assert np.linalg.norm(th[i, t] - want[t]) <= (1e-10 * kappa + 1e-13) * n
            assert np.linalg.norm(th0[i, t] - want[t]) <= 4 * 2.0 ** -24 * kappa * n
