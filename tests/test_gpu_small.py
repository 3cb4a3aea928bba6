"""Systems of one and two block columns: refinement in one launch, at the edges of its sizes and columns."""
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


# N = (2m + 1)^d: 3, 63, 65, 127 and 121 unknowns (one and two block columns); 129 unknowns or 5 targets take the other path
@pytest.mark.parametrize("d,m,nlam,T", [(1, 1, 1, 1), (1, 31, 3, 4), (1, 32, 1, 2), (1, 63, 7, 1), (1, 63, 2, 3),
                                        (2, 5, 300, 4), (1, 64, 2, 4), (1, 63, 2, 5)])
def test_small_solves(fk, d, m, nlam, T):
    import torch
    rng = np.random.default_rng(1000 * m + nlam)
    X = rng.uniform(-np.pi, np.pi, (d, 3000))
    X = X + 0.5 * np.sin(X)
    Y = rng.standard_normal((T, 3000))
    M, b = oracle.gram_generator(X, m), oracle.rhs(X, Y, m)
    lams = list(10.0 ** np.linspace(-4, -1, nlam))
    p = oracle.sobolev_weights(m, d, 1.0)
    args = (torch.from_numpy(M).cuda(), torch.from_numpy(b).cuda(), m, lams)
    th, info = fk.solve(*args, penalty="sobolev", s=1.0, ctx=fk.Context(0), info=True)
    assert 1 <= info["refine_iters"] <= 2
    # one unrefined solve: FP32-class, kappa(A) 2^-24 with a factor for the sums over N terms
    th0, info0 = fk.solve(*args, penalty="sobolev", s=1.0, ctx=fk.Context(0, max_refine=0, refine_tol=1e-2), info=True)
    assert info0["refine_iters"] == 0
    # steps that are checked one by one
    th1 = fk.solve(*args, penalty="sobolev", s=1.0, ctx=fk.Context(0, max_refine=5, refine_tol=2e-8))
    th, th0, th1 = th.cpu().numpy(), th0.cpu().numpy(), th1.cpu().numpy()
    for i in sorted({0, nlam - 1}):
        A = oracle.system_matrix(M, m, lams[i], p)
        want = oracle.solve_system(A, b)
        kappa = np.linalg.cond(A)
        for t in range(T):
            n = np.linalg.norm(want[t])
            assert np.linalg.norm(th[i, t] - want[t]) <= (1e-10 * kappa + 1e-13) * n
            assert np.linalg.norm(th1[i, t] - want[t]) <= (2e-8 * kappa + 1e-13) * n
            assert np.linalg.norm(th0[i, t] - want[t]) <= 4 * 2.0 ** -24 * kappa * n
    bad = b.copy()
    bad[T - 1, 0] = np.nan
    with pytest.raises(fk.FkError):
        fk.solve(args[0], torch.from_numpy(bad).cuda(), m, lams, penalty="sobolev", s=1.0)
