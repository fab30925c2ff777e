"""Truncated SVDs of blocks whose norms square out of the range of FP64.  Rows
that small or large have always counted as orthogonal, so such a block is taken
as it stands; every size has to see it that way when it decides whether to
iterate on."""
import numpy as np
import pytest

from helpers import pl, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pre", [0, 1])
@pytest.mark.parametrize("scale", [1e-150, 1e-100, 1e-85, 1.0, 1e100])
@pytest.mark.parametrize("nr,nc", [(40, 40), (64, 70), (65, 66), (100, 90), (200, 300)])
def test_extreme_scales_are_accepted(nr, nc, scale, pre):
    ctx = pl.Context(0)
    rng = np.random.default_rng(nr)
    M = rng.standard_normal((nr, nc)) * np.logspace(0, -4, nr)[:, None]
    M *= scale / np.linalg.norm(M)
    pl.set_svd_precondition(ctx, pre)
    res = pl.SvdResult(ctx, pl.Bond({0: nr}), pl.Bond({2: nc}), pl.Phys((-1, 1)), dev(M.reshape(-1)), 10 ** 6,
                       mode=pl.ABSORB_RIGHT)
    assert res.code == 0                    # no block ran out of sweeps
    assert res.lam.size > 0 and np.all(np.isfinite(res.lam))
    if scale == 1.0:
        ref = np.linalg.svd(M, compute_uv=False)
        assert np.max(np.abs(np.sort(res.lam)[::-1] - ref[:res.lam.size])) <= 1e-13
    ctx.close()
