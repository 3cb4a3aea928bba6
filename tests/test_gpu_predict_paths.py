"""Prediction by direct sums and from the LDS-resident grid, at the edges of their splits."""
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


def _theta(rng, T, d, m):
    N = (2 * m + 1) ** d
    c = rng.standard_normal((T, N)) + 1j * rng.standard_normal((T, N))
    return 0.5 * (c + c[:, ::-1].conj())


def _run(fk, th, Xq, m):
    import torch
    return fk.predict(torch.from_numpy(th).cuda(), torch.from_numpy(Xq).cuda(), m).cpu().numpy()


# 8 points per workgroup; 5, 9 or 17 modes of the last axis per lane
@pytest.mark.parametrize("d,m,T,nq", [(1, 1, 1, 1), (1, 64, 3, 9), (2, 19, 1, 7), (2, 20, 2, 8), (2, 35, 1, 9),
                                      (2, 36, 1, 17), (2, 64, 1, 3), (3, 3, 2, 15), (3, 16, 1, 9)])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_direct_sums(fk, d, m, T, nq, dtype):
    rng = np.random.default_rng(d * 1000 + m + nq)
    th = _theta(rng, T, d, m)
    Xq = rng.uniform(-2 * np.pi, 2 * np.pi - 1e-6, (d, nq)).astype(dtype)
    f = _run(fk, th, Xq, m)
    want = np.stack([oracle.predict(th[t][None], Xq.astype(np.float64), m).real[0] for t in range(T)])
    # FP64 sums of N terms (1e-13 of the sum of moduli), rounded to FP32 (6e-8)
    assert (np.abs(f - want) <= 6.1e-8 * np.abs(want) + 1e-13 * np.abs(th).sum(axis=1, keepdims=True)).all()


# chunks of 4096, 2048 and 1024 points; all sets or one per workgroup; points whose windows start in one
# bank (more than a bank's share of slots); the largest grid that stays in LDS
@pytest.mark.parametrize("m,T,nq,shape", [(8, 16, 65_537, "flat"), (8, 16, 65_536, "one"), (16, 3, 200_001, "flat"),
                                          (20, 1, 40_001, "flat"), (20, 1, 40_001, "one"), (41, 2, 90_001, "flat")])
def test_grid_in_lds(fk, m, T, nq, shape):
    rng = np.random.default_rng(m + nq)
    th = _theta(rng, T, 2, m)
    Xq = rng.uniform(-np.pi, np.pi, (2, nq))
    if shape == "one":
        Xq[:, 11:] = 0.7 + 1e-4 * Xq[:, 11:]
    Xq = Xq.astype(np.float32)
    f = _run(fk, th, Xq, m)
    # every point of a sample against the direct sums: kernel error 2e-7 per axis and FP32 sums
    pick = np.unique(np.concatenate([np.arange(12), rng.integers(0, nq, 400), [nq - 1, 4095, 4096, 1023, 1024]]))
    want = np.stack([oracle.predict(th[t][None], Xq[:, pick].astype(np.float64), m).real[0] for t in range(T)])
    assert (np.abs(f[:, pick] - want) <= 1e-6 * np.abs(th).sum(axis=1, keepdims=True)).all()
    assert np.isfinite(f).all()


@pytest.mark.parametrize("nq", [5, 70_000])
def test_out_of_range_is_reported(fk, nq):
    Xq = np.zeros((2, nq), dtype=np.float32)
    Xq[1, nq - 1] = 7.0
    th = np.ones((1, 17 * 17), dtype=np.complex128)
    with pytest.raises(fk.FkError) as e:
        _run(fk, th, Xq, 8)
    assert e.value.code == 2
