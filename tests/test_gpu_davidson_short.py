"""Davidson runs on vectors short enough that one workgroup does a step's passes
(up to 4096 elements: 1, 2 or up to 4 a thread) and just past that, with subspaces
that restart often and up to the largest that the joint passes take, against the
oracle's iteration on the same H_eff.  Both stop at a residual of 1e-9, so the
energies differ by its square over the gap and by rounding: 1e-9 |E| is wide."""
import pytest

from helpers import pl, tables, blocks_to_flat, flat_to_blocks, mpo_site, dev, host, say
from oracle import dmrg
from oracle.blocks import Bond, two_site_keys, two_site_shape, flatten, unflatten
from test_gpu_core import _hermitian_problem

pytestmark = pytest.mark.gpu
PQ = (-1, 1)


@pytest.mark.parametrize("N,m,sub,prec,n", [(4, 2, 3, pl.F64, 6), (14, 24, 4, pl.F64, 528), (14, 37, 8, pl.F32, 1122),
                                            (14, 50, 8, pl.F64, 2066), (14, 64, 16, pl.F32, 3432),
                                            (16, 68, 5, pl.F64, 3726), (16, 74, 8, pl.F64, 4212)])
def test_davidson_on_short_vectors(N, m, sub, prec, n):
    import torch
    assert torch.cuda.is_available()
    ctx = pl.Context(0)
    c = N // 2 - 1
    mpo, bonds, Lo, Ro, Lg, Rg, psi = _hermitian_problem(ctx, N, m, 3, c)
    bl, br = Bond(bonds[c]), Bond(bonds[c + 2])
    keys = two_site_keys(bl, br, PQ)
    shapes = [two_site_shape(k, bl, br, PQ) for k in keys]
    mv = lambda v: flatten(dmrg.heff_apply(Lo, Ro, mpo.W[c], mpo.W[c + 1], unflatten(v, keys, shapes),
                                           bl, br, PQ, mpo.deltas[c], mpo.deltas[c + 2]), keys, shapes)
    diag = flatten(dmrg.heff_diag(Lo, Ro, mpo.W[c], mpo.W[c + 1], bl, br, PQ, mpo.deltas[c], mpo.deltas[c + 2]),
                   keys, shapes)
    x0 = flatten(psi, keys, shapes)
    assert x0.size == n
    Eo, xo, rno, nmvo = dmrg.davidson(mv, x0, diag, dmrg.DavidsonParams(400, 1e-9, sub))
    t, (B1, B2, P) = tables(bonds[c], bonds[c + 2], PQ, mpo.deltas[c], mpo.deltas[c + 2])
    W1, W2 = mpo_site(mpo, c), mpo_site(mpo, c + 1)
    op = pl.Heff(ctx, B1, B2, P, W1, W2, Lg, Rg, prec)
    op64 = pl.Heff(ctx, B1, B2, P, W1, W2, Lg, Rg, pl.F64) if prec != pl.F64 else None
    x = dev(blocks_to_flat(psi, t["x"][0], t["x"][1], pl.TWO_SITE))
    E, rn, nmv, code = pl.davidson_step(ctx, op, x, max_matvec=400, max_sub=sub, tol=1e-9, op64=op64)
    say("n", n, "max_sub", sub, "E", E, "oracle", Eo, "resid", rn, "products", nmv, "oracle", nmvo)
    assert rno <= 1e-9 and code == 0
    assert abs(E - Eo) <= 1e-9 * abs(Eo)
    xg = flatten(flat_to_blocks(host(x), t["x"][0], pl.TWO_SITE), keys, shapes)
    assert abs(abs(xg @ xo) - 1.0) <= 1e-6
    ctx.close()
