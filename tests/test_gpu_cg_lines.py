"""Line transforms that share a wave: each length, with a last workgroup that is not full, and skipped systems."""
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


# lines of 8, 16, 32, 64, 128 and 512 points; odd numbers of lines
@pytest.mark.parametrize("d,m", [(1, 1), (2, 1), (2, 2), (2, 5), (2, 15), (2, 31), (2, 64), (3, 1), (3, 3), (3, 7),
                                 (3, 9)])
def test_line_lengths(fk, d, m):
    import torch
    rng = np.random.default_rng(10 * d + m)
    n, V = (60, 3) if m < 64 else (20, 1)
    M = oracle.gram_generator(rng.uniform(-np.pi, np.pi, (d, n)), m)
    N = (2 * m + 1) ** d
    x = rng.standard_normal((V, N)) + 1j * rng.standard_normal((V, N))
    y = fk.toeplitz_apply(torch.from_numpy(M).cuda(), torch.from_numpy(x).cuda(), m).cpu().numpy()
    rows = np.unique(np.concatenate([[0, N // 2, N - 1], rng.choice(N, min(N, 30), replace=False)]))
    for v in range(V):
        ref = oracle.toeplitz_apply_rows(M, x[v], m, rows)
        # FP64 transforms: a few ulp per level of the largest entry
        np.testing.assert_allclose(y[v, rows], ref, rtol=0, atol=1e-12 * max(np.abs(ref).max(), np.abs(y[v]).max()))


# systems that leave the iteration at different times, 125 and 3375 unknowns (256 and 1024 threads per system)
@pytest.mark.parametrize("m", [2, 7])
def test_3d_systems(fk, m):
    import torch
    rng = np.random.default_rng(m)
    X = rng.uniform(-np.pi, np.pi, (3, 4000))
    Y = rng.standard_normal((2, 4000))
    M, b = oracle.gram_generator(X, m), oracle.rhs(X, Y, m)
    b[1] = 0.0
    lams = [1.0, 1e-1, 1e-3]
    th, inf = fk.solve_cg(torch.from_numpy(M).cuda(), torch.from_numpy(b).cuda(), m, lams, penalty="sobolev", s=2.0,
                          tol=1e-11, maxit=2000, info=True)
    p = oracle.sobolev_weights(m, 3, 2.0)
    for i, lam in enumerate(lams):
        A = oracle.system_matrix(M, m, lam, p)
        y = th[i, 0].cpu().numpy()
        assert np.linalg.norm(b[0] - A @ y) <= 2e-11 * np.linalg.norm(b[0])   # stopped at 1e-11
        assert float(th[i, 1].abs().max()) == 0.0 and inf["relres"][i][1] == 0.0
