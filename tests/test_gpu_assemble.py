"""Assembly of the real system by pairs of rows and columns: padding edges, constant row, box operators."""
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


# N = (2m + 1)^d against the padding to 64: 3, 63 (one row of padding), 65 (63 rows), 129, 9, 49, 225; the
# refined residual is at most 1e-10, so the solution is within kappa(A) 1e-10 of the system's
@pytest.mark.parametrize("d,m", [(1, 1), (1, 31), (1, 32), (1, 64), (2, 1), (2, 3), (2, 7)])
@pytest.mark.parametrize("box", [False, True])
def test_assembled_systems(fk, d, m, box):
    import torch
    rng = np.random.default_rng(10 * m + d)
    n, lam, mu = 2000, 1e-2, 1e-3
    X = rng.uniform(-1.0, 1.2, (d, n))
    Y = rng.standard_normal((1, n))
    M, b = oracle.gram_generator(X, m), oracle.rhs(X, Y, m)
    kw = dict(penalty="sobolev", s=1.0)
    if box:
        alpha = [[1], [0]] if d == 1 else [[1, 1], [0, 2], [1, 0], [0, 0]]
        coef = [1.0, 1.0] if d == 1 else [1.0, 0.5, 1.0, -2.0]
        lo, hi = (-1.0, -0.3)[:d], (0.5, 1.2)[:d]
        Q = oracle.piml_box_penalty(m, d, lam, mu, oracle.pde_symbol(m, d, alpha, coef), lo, hi, s=1.0)
        A = oracle.system_matrix(M, m, 0.0, Q)
        kw = dict(penalty="pde_box", s=1.0, mu=mu, alpha=alpha, coef=coef, box_lo=lo, box_hi=hi)
    else:
        A = oracle.system_matrix(M, m, lam, oracle.sobolev_weights(m, d, 1.0))
    th = fk.solve(torch.from_numpy(M).cuda(), torch.from_numpy(b).cuda(), m, [lam], ctx=fk.Context(0), **kw)
    want = oracle.solve_system(A, b)
    assert np.linalg.norm(th[0].cpu().numpy() - want) <= (1e-10 * np.linalg.cond(A) + 1e-13) * np.linalg.norm(want)
