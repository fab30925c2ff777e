"""An operator on bonds that no pair of local states connects: its vectors are
empty, products with it do nothing, and a Davidson run returns at once with
energy 0, whatever its subspace."""
import pytest

from helpers import pl, mpo_site, say
from oracle import models, mpo as M

pytestmark = pytest.mark.gpu
PQ = (-1, 1)


@pytest.mark.parametrize("sub", [2, 8, 16, 17])
@pytest.mark.parametrize("prec", [pl.F64, pl.F32])
def test_davidson_on_an_empty_tensor(prec, sub):
    import torch
    mpo = M.build_mpo(models.heisenberg_terms(models.chain_bonds(8)), 8, models.OPS, PQ)
    c = 3
    B1, B2, P = pl.Bond({0: 3}), pl.Bond({6: 2}), pl.Phys(PQ)
    assert pl.layout(pl.TWO_SITE, B1, B2, P)[1] == 0
    ctx = pl.Context(0)
    mk = lambda n: torch.zeros(max(n, 1), dtype=torch.float64, device="cuda")
    L = mk(pl.layout(pl.ENV_L, B1, deltas=mpo.deltas[c])[1])
    R = mk(pl.layout(pl.ENV_R, B2, deltas=mpo.deltas[c + 2])[1])
    op = pl.Heff(ctx, B1, B2, P, mpo_site(mpo, c), mpo_site(mpo, c + 1), L, R, prec)
    op64 = pl.Heff(ctx, B1, B2, P, mpo_site(mpo, c), mpo_site(mpo, c + 1), L, R, pl.F64) if prec != pl.F64 else None
    x = mk(0)
    E, rn, nmv, code = pl.davidson_step(ctx, op, x, max_matvec=6, max_sub=sub, tol=1e-10, op64=op64)
    say("E", E, "resid", rn, "products", nmv)
    assert (E, rn, code) == (0.0, 0.0, 0) and nmv in (1, 2)
    assert float(x[0]) == 0.0
    ctx.close()
