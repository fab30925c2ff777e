"""GPU block-Jacobi SVD at the sizes where its kernels change: the one-workgroup
instances (rows up to 16, 32, 64), the padding of the 64-row pairs, one and
several rounds, odd and ragged blocks, rank-deficient ones; against LAPACK's
SVD of the same dense block."""
import numpy as np
import pytest

from helpers import pl, dev, host

pytestmark = pytest.mark.gpu
PQ = (-1, 1)


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    c = pl.Context(0)
    yield c
    c.close()


def _block(nr, nc, seed, rank=None):
    """A graded nr x nc block (rows and columns weighted over four decades), of the given rank."""
    rng = np.random.default_rng(seed)
    k = min(nr, nc) if rank is None else rank
    if rank is None:
        M = rng.standard_normal((nr, nc))
    else:
        M = rng.standard_normal((nr, k)) @ rng.standard_normal((k, nc))
    M *= np.logspace(0, -4, nr)[:, None] * np.logspace(0, -4, nc)[rng.permutation(nc)][None, :]
    return M / np.linalg.norm(M)


SIZES = [(1, 1), (2, 3), (15, 15), (16, 40), (17, 16), (31, 33), (32, 32), (33, 70), (63, 64), (64, 64), (64, 200),
         (65, 65), (96, 65), (127, 130), (128, 128), (129, 300), (191, 192), (257, 193)]


@pytest.mark.parametrize("pre", [0, 1])
@pytest.mark.parametrize("nr,nc,rank", [s + (None,) for s in SIZES] + [(20, 30, 3), (64, 64, 1), (100, 90, 40)])
def test_block_svd_sizes(ctx, nr, nc, rank, pre):
    """One middle-charge block.  A backward-stable SVD leaves singular values
    within a few hundred eps of lambda_1 = O(1) and factors orthonormal to a
    few hundred eps at these sizes: 1e-13 and 1e-12."""
    M = _block(nr, nc, 7 * nr + nc, rank)
    B1, B2, P = pl.Bond({0: nr}), pl.Bond({2: nc}), pl.Phys(PQ)
    x = dev(M.reshape(-1))
    pl.set_svd_precondition(ctx, pre)
    try:
        res = pl.SvdResult(ctx, B1, B2, P, x, 10 ** 6, cutoff=1e-13, eps=1e-4, mode=pl.ABSORB_RIGHT)
    finally:
        pl.set_svd_precondition(ctx, 1)
    assert res.code == 0
    ref = np.linalg.svd(M, compute_uv=False)
    k = sum(res.bond.values())
    assert list(res.bond) == [1] and (rank is None or k == rank)
    assert np.max(np.abs(np.sort(res.lam)[::-1] * np.sqrt(np.sum(ref[:k] ** 2)) - ref[:k])) <= 1e-13 * ref[0]
    A, B, R = host(res.A).reshape(nr, k), host(res.B).reshape(k, nc), host(res.right).reshape(k, nc)
    assert np.abs(A.T @ A - np.eye(k)).max() <= 1e-12
    assert np.abs(B @ B.T - np.eye(k)).max() <= 1e-12
    assert np.linalg.norm(A @ R - M) <= 1e-12


def test_zero_rows_and_columns(ctx):
    """Blocks with vanishing rows and columns keep the other singular values."""
    M = _block(80, 70, 3)
    M[10:25] = 0.0
    M[:, 40:] = 0.0
    x = dev(M.reshape(-1))
    res = pl.SvdResult(ctx, pl.Bond({0: 80}), pl.Bond({2: 70}), pl.Phys(PQ), x, 10 ** 6, cutoff=1e-13,
                       mode=pl.ABSORB_LEFT)
    ref = np.linalg.svd(M, compute_uv=False)
    k = sum(res.bond.values())
    assert k == 40
    assert np.max(np.abs(res.lam * np.linalg.norm(ref) - ref[:k])) <= 1e-13 * ref[0]
    assert np.linalg.norm(host(res.left).reshape(80, k) @ host(res.B).reshape(k, 70) * np.linalg.norm(ref) - M) <= 1e-12
