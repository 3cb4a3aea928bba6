"""Prediction from grids in memory: each line length of the transforms, a wave per point, and its last waves."""
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


# d = 3: grids of 16 to 256 cells per axis; d = 1: lines of 16 to 512 points; d = 2, m = 64: past the grids in LDS.
# Points of one to four workgroups of 16 (4 points a wave) and more; one point in the last wave.
@pytest.mark.parametrize("d,m,T,nq", [(3, 1, 1, 20_001), (3, 3, 3, 20_001), (3, 5, 2, 16_385), (3, 9, 1, 8_193),
                                      (3, 20, 1, 5_003), (3, 31, 2, 4_097), (3, 12, 17, 2_049), (2, 64, 1, 30_001),
                                      (2, 64, 3, 270_017), (1, 1, 1, 70_001), (1, 9, 3, 70_001), (1, 33, 2, 70_001),
                                      (1, 64, 5, 70_001)])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_from_grids(fk, d, m, T, nq, dtype):
    import torch
    rng = np.random.default_rng(100 * d + m)
    N = (2 * m + 1) ** d
    c = rng.standard_normal((T, N)) + 1j * rng.standard_normal((T, N))
    th = 0.5 * (c + c[:, ::-1].conj())
    Xq = rng.uniform(-np.pi, np.pi, (d, nq)).astype(dtype)
    Xq[:, :4] = np.array([-np.pi, 3.1415925, 0.0, 1e-7])
    Xq[:, 4:12] += np.where(rng.random((d, 8)) < 0.5, 2.5, -2.5).astype(dtype)   # outside [-pi, pi), folded
    f = fk.predict(torch.from_numpy(th).cuda(), torch.from_numpy(Xq).cuda(), m).cpu().numpy()
    pick = np.unique(np.concatenate([np.arange(80), rng.integers(0, nq, 60), np.arange(nq - 20, nq)]))
    want = oracle.predict(th, Xq[:, pick].astype(np.float64), m).real
    # kernel error 2e-7 per axis and FP32 sums, of the sum of moduli
    assert (np.abs(f[:, pick] - want) <= 2e-6 * np.abs(th).sum(axis=1, keepdims=True)).all()
    assert np.isfinite(f).all()


@pytest.mark.parametrize("d,m,nq", [(3, 8, 9_001), (2, 64, 40_001)])
def test_bad_points(fk, d, m, nq):
    import torch
    rng = np.random.default_rng(1)
    th = torch.ones((1, (2 * m + 1) ** d), dtype=torch.complex128, device="cuda")
    for bad in (np.nan, 7.0, -np.inf):
        Xq = rng.uniform(-np.pi, np.pi, (d, nq)).astype(np.float32)
        Xq[d - 1, nq - 1] = bad
        with pytest.raises(fk.FkError):
            fk.predict(th, torch.from_numpy(Xq).cuda(), m)
