"""Conjugate gradients with one workgroup per system: edges of its sizes, of its launches, and its stops."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-11


@pytest.fixture(scope="module")
def fk():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2509_02649_amd as fk
    return fk


def _case(d, m, T, n, seed, half=np.pi):
    rng = np.random.default_rng(seed)
    X = rng.uniform(-half, half, (d, n))
    X = X + 0.4 * np.sin(X)
    Y = rng.standard_normal((T, n))
    return oracle.gram_generator(X, m), oracle.rhs(X, Y, m)


def _dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


# d = 2: 7 and 33 take the passes; 8 the smallest; 16 and 32 (lags +-2m share a position of the 64 and of the 128
# points) and their neighbours.  d = 1: lines of 8, 128, 256 (exactly 4m + 1 = 253), 512 and 1024 points.
@pytest.mark.parametrize("d,m", [(2, 7), (2, 8), (2, 15), (2, 16), (2, 17), (2, 31), (2, 32), (2, 33),
                                 (1, 1), (1, 31), (1, 63), (1, 64), (1, 255)])
@pytest.mark.parametrize("colloc", [False, True])
def test_sizes(fk, d, m, colloc):
    T, lams, mu = 2, [1e-1, 1e-3], 1e-4
    M, b = _case(d, m, T, 3000, m)
    p = oracle.sobolev_weights(m, d, 2.0)
    kw, C = {}, 0.0
    if colloc:
        Mr, _ = _case(d, m, 1, 500, m + 1, 1.5)
        D = oracle.pde_symbol(m, d, [[1] * d, [0] * d], [1.0, 0.5])
        S = oracle.system_matrix(Mr, m, 0.0, p)
        C = mu * (np.conj(D)[:, None] * S * D[None, :])
        kw = dict(collocation=(mu, _dev(Mr), _dev(D)))
    th, inf = fk.solve_cg(_dev(M), _dev(b), m, lams, penalty="sobolev", s=2.0, tol=TOL, maxit=3000, info=True, **kw)
    th = th.cpu().numpy()
    for i, lam in enumerate(lams):
        A = oracle.system_matrix(M, m, lam, p) + C
        for t in range(T):
            res = np.linalg.norm(b[t] - A @ th[i, t]) / np.linalg.norm(b[t])
            # stopped at a recursive residual of TOL; what rounding adds to the true one is far below it
            assert res <= 2 * TOL and inf["relres"][i][t] <= 2 * TOL, (lam, t, res, inf["relres"][i][t])


# 2048 systems run 32 iterations a launch: systems that end in the first launch, and in later ones
@pytest.mark.parametrize("d,m", [(1, 40), (2, 8)])
def test_several_launches(fk, d, m):
    T = 2
    lams = list(10.0 ** np.linspace(-9, 1, 1024))
    M, b = _case(d, m, T, 3000, 5)
    b[1] = 0.0                                  # a system that is solved before it starts
    p = oracle.sobolev_weights(m, d, 2.0)
    th, inf = fk.solve_cg(_dev(M), _dev(b), m, lams, penalty="sobolev", s=2.0, tol=TOL, maxit=3000, info=True)
    th = th.cpu().numpy()
    print("iterations", inf["iters"])
    for i in (0, 1, 500, 1023):
        A = oracle.system_matrix(M, m, lams[i], p)
        assert np.linalg.norm(b[0] - A @ th[i, 0]) <= 2 * TOL * np.linalg.norm(b[0])
    assert np.all(th[:, 1] == 0.0) and max(r[1] for r in inf["relres"]) == 0.0
    # the same systems, a few at a time (one launch)
    few = fk.solve_cg(_dev(M), _dev(b), m, lams[:3], penalty="sobolev", s=2.0, tol=TOL, maxit=3000).cpu().numpy()
    assert np.array_equal(few, th[:3])


# with the collocation term, 64 systems take four launches per iteration and 65 one workgroup each
@pytest.mark.parametrize("m", [17, 32])
def test_many_collocation_systems(fk, m):
    mu = 1e-4
    M, b = _case(2, m, 1, 3000, 8)
    Mr, _ = _case(2, m, 1, 500, 9, 1.5)
    D = oracle.pde_symbol(m, 2, [[1, 1], [0, 0]], [1.0, 0.5])
    lams = list(10.0 ** np.linspace(-4, 0, 65))
    kw = dict(penalty="sobolev", s=2.0, tol=TOL, maxit=3000, info=True, collocation=(mu, _dev(Mr), _dev(D)))
    th, inf = fk.solve_cg(_dev(M), _dev(b), m, lams, **kw)
    few, inf64 = fk.solve_cg(_dev(M), _dev(b), m, lams[:64], **kw)
    p = oracle.sobolev_weights(m, 2, 2.0)
    C = mu * (np.conj(D)[:, None] * oracle.system_matrix(Mr, m, 0.0, p) * D[None, :])
    S = oracle.system_matrix(M, m, 0.0, p) + C
    for i in (0, 40, 63):
        for x in (th, few):
            y = x[i, 0].cpu().numpy()
            assert np.linalg.norm(b[0] - S @ y - lams[i] * p * y) <= 2 * TOL * np.linalg.norm(b[0])
    assert max(r[0] for r in inf["relres"]) <= 2 * TOL and max(r[0] for r in inf64["relres"]) <= 2 * TOL
    assert abs(inf["iters"] - inf64["iters"]) <= 1


def test_stops_with_collocation(fk):
    m = 20
    M, b = _case(2, m, 1, 3000, 3)
    Mr, _ = _case(2, m, 1, 500, 9, 1.5)
    col = (1e-4, _dev(Mr), _dev(oracle.pde_symbol(m, 2, [[1, 0], [0, 0]], [1.0, 0.5])))
    for bad in (np.nan, np.inf):
        c = b.copy()
        c[0, 7] = bad
        with pytest.raises(fk.FkError):
            fk.solve_cg(_dev(M), _dev(c), m, [1e-3], collocation=col)
    neg = Mr.copy()
    neg[2 * m, 2 * m] = -1.0                    # the diagonal of Sigma_r
    with pytest.raises(fk.FkError):
        fk.solve_cg(_dev(M), _dev(b), m, [1e-3], collocation=(1e-4, _dev(neg), col[2]))
    ind = np.zeros_like(M)
    ind[2 * m, 2 * m], ind[2 * m, 2 * m + 1], ind[2 * m, 2 * m - 1] = 1.0, 4.0, 4.0
    with pytest.raises(fk.FkError):
        fk.solve_cg(_dev(ind), _dev(b), m, [1e-6], collocation=(1e-12, col[1], col[2]))
    with pytest.raises(fk.FkError):             # iteration limit
        fk.solve_cg(_dev(M), _dev(b), m, [1e-5], maxit=9, tol=1e-12, collocation=col)
    th, inf = fk.solve_cg(_dev(M), _dev(0.0 * b), m, [1e-3], info=True, collocation=col)
    assert inf["iters"] == 0 and float(th.abs().max()) == 0.0 and inf["relres"] == [[0.0]]


def test_stops(fk):
    M, b = _case(2, 16, 1, 3000, 3)
    for bad in (np.nan, np.inf):
        c = b.copy()
        c[0, 7] = bad
        with pytest.raises(fk.FkError):
            fk.solve_cg(_dev(M), _dev(c), 16, [1e-3])
    neg = M.copy()
    neg[32, 32] = -1.0                          # the diagonal of Sigma
    with pytest.raises(fk.FkError):
        fk.solve_cg(_dev(neg), _dev(b), 16, [1e-3])
    ind = np.zeros_like(M)
    ind[32, 32], ind[32, 33], ind[32, 31] = 1.0, 4.0, 4.0   # Hermitian, not positive definite
    with pytest.raises(fk.FkError):
        fk.solve_cg(_dev(ind), _dev(b), 16, [1e-6])
    with pytest.raises(fk.FkError):             # iteration limit
        fk.solve_cg(_dev(M), _dev(b), 16, [1e-5], maxit=3)
