"""Truncated SVDs of blocks with few but long rows, where the one-workgroup
iteration takes its Gram sums by all waves (1024 columns, up to 16 rows) and where
it gives way to the sweeps of many launches with partial Gram sums; wide and
tall, against LAPACK's SVD of the same block."""
import numpy as np
import pytest

from helpers import pl, dev, host

pytestmark = pytest.mark.gpu
SIZES = [(1, 3000), (1, 6001), (2, 1023), (2, 1024), (5, 1025), (8, 5999), (16, 1040), (16, 6000), (16, 6001), (3, 9000),
         (17, 3000), (17, 3001), (31, 4111), (32, 2999), (33, 1400), (33, 1401), (48, 4096), (63, 1401), (64, 2049),
         (64, 1500)]


@pytest.mark.parametrize("tall", [False, True])
@pytest.mark.parametrize("nv,length", SIZES)
def test_few_long_rows(nv, length, tall):
    """The bars of the other block sizes: singular values to 1e-13 of the largest,
    factors orthonormal to 1e-12."""
    rng = np.random.default_rng(nv * length)
    M = rng.standard_normal((nv, length)) * np.logspace(0, -4, nv)[:, None]
    M *= np.logspace(0, -4, length)[rng.permutation(length)][None, :]
    if nv == 48:
        M[40:] = M[:8]                      # rank 40
    M /= np.linalg.norm(M)
    if tall:
        M = np.ascontiguousarray(M.T)
    nr, nc = M.shape
    ctx = pl.Context(0)
    pl.set_svd_precondition(ctx, 0 if length < 2048 else 1)
    res = pl.SvdResult(ctx, pl.Bond({0: nr}), pl.Bond({2: nc}), pl.Phys((-1, 1)), dev(M.reshape(-1)), 10 ** 6,
                       cutoff=1e-13, mode=pl.ABSORB_RIGHT)
    assert res.code == 0
    ref = np.linalg.svd(M, compute_uv=False)
    k = sum(res.bond.values())
    assert k == (40 if nv == 48 else nv)
    assert np.max(np.abs(np.sort(res.lam)[::-1] * np.sqrt(np.sum(ref[:k] ** 2)) - ref[:k])) <= 1e-13 * ref[0]
    A, B, R = host(res.A).reshape(nr, k), host(res.B).reshape(k, nc), host(res.right).reshape(k, nc)
    assert np.abs(A.T @ A - np.eye(k)).max() <= 1e-12
    assert np.abs(B @ B.T - np.eye(k)).max() <= 1e-12
    assert np.linalg.norm(A @ R - M) <= 1e-12
    ctx.close()
