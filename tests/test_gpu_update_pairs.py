"""The factorization with two pairs of block columns per update, and its last columns."""
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


# nb = 67 and 63 block columns: an odd one out, and groups that end one and two pairs before the last column; 16
# lambdas take two pairs per update, 2 take one
@pytest.mark.parametrize("m,nlam", [(32, 16), (31, 16)])
def test_groups_of_pairs(fk, m, nlam):
    import torch
    rng = np.random.default_rng(m)
    X = rng.uniform(-np.pi, np.pi, (2, 20_000))
    X = X + 0.3 * np.sin(X)
    Y = rng.standard_normal((1, 20_000))
    M, b = oracle.gram_generator(X, m), oracle.rhs(X, Y, m)
    lams = list(10.0 ** np.linspace(-4, -1, nlam))
    args = (torch.from_numpy(M).cuda(), torch.from_numpy(b).cuda(), m)
    th, info = fk.solve(*args, lams, penalty="sobolev", s=1.0, info=True)
    assert info["refine_iters"] <= 2
    two = fk.solve(*args, [lams[0], lams[-1]], penalty="sobolev", s=1.0)
    # the residual of both is at most 1e-10 (the refinement's tolerance); kappa(A) <= (M0 + lam p) / lam <= 2e4
    for i, j in ((0, 0), (nlam - 1, 1)):
        d = torch.linalg.norm(th[i] - two[j]) / torch.linalg.norm(two[j])
        assert float(d) <= 2 * 2e4 * 1e-10
    # one unrefined solve: a mistake in the factor would show at once
    th0 = fk.solve(*args, lams, penalty="sobolev", s=1.0, ctx=fk.Context(0, max_refine=0, refine_tol=1e-2))
    assert float(torch.linalg.norm(th0 - th) / torch.linalg.norm(th)) <= 4 * 2.0 ** -24 * 2e4
