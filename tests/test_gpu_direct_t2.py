"""H_eff products whose stage 1 writes the W stage's one-term blocks itself (T1 of
32 MB and more): every kernel that does so, on ragged sectors and an MPO whose
entries are sums of one and of several terms with coefficients other than 1,
against the same contraction on dense NumPy blocks."""
import numpy as np
import pytest

from helpers import pl, synth, blocks_to_flat, dev, host, mpo_site
from oracle import models, dmrg, mpo as M
from oracle.blocks import Bond

pytestmark = pytest.mark.gpu
PQ = (-1, 1)
SITE = 5
BL, BR = {-3: 61, -1: 331, 1: 340, 3: 55}, {-3: 40, -1: 353, 1: 324, 3: 71}


@pytest.fixture(scope="module")
def problem():
    import torch
    assert torch.cuda.is_available()
    bonds = models.square_cylinder_bonds(3, 4)
    mpo = M.build_mpo(models.heisenberg_terms(bonds), 12, models.OPS, PQ)
    rng = np.random.default_rng(1)
    W1, W2 = (np.array(mpo.W[i], dtype=float) for i in (SITE, SITE + 1))
    W1 *= np.where(W1 == 1.0, 1.0, rng.uniform(0.5, 2.0, W1.shape))
    dl, dr = mpo.deltas[SITE], mpo.deltas[SITE + 2]
    L, R = synth.random_env_blocks(BL, dl, rng), synth.random_env_blocks(BR, dr, rng)
    psi = synth.random_two_site_blocks(BL, BR, PQ, rng)
    B1, B2, P = pl.Bond(BL), pl.Bond(BR), pl.Phys(PQ)
    tx, nx = pl.layout(pl.TWO_SITE, B1, B2, P)
    tl, nl = pl.layout(pl.ENV_L, B1, deltas=dl)
    tr, nr = pl.layout(pl.ENV_R, B2, deltas=dr)
    ref = dmrg.heff_apply(L, R, W1, W2, psi, Bond(BL), Bond(BR), PQ, dl, dr)
    args = (B1, B2, P, pl.MpoSite(W1, dl, mpo.deltas[SITE + 1]), pl.MpoSite(W2, mpo.deltas[SITE + 1], dr),
            dev(blocks_to_flat(L, tl, nl, pl.ENV_L)), dev(blocks_to_flat(R, tr, nr, pl.ENV_R)))
    return args, dev(blocks_to_flat(psi, tx, nx, pl.TWO_SITE)), blocks_to_flat(ref, tx, nx, pl.TWO_SITE)


# staged, LDS-DMA, register-direct and quad kernels
@pytest.mark.parametrize("prec,shape", [("f64", s) for s in (None, 0, 1, 2, 3, 4, 5, 8, 9, 10, 11, 12, 13, 14)] +
                         [("f32", s) for s in (None, 3, 4, 5, 6, 7, 8, 9, 10, 15, 16, 17, 18)] +
                         [("bf16x3", s) for s in (None, 8, 9, 10, 15, 16, 17, 18)])
def test_one_term_blocks_from_stage_1(problem, prec, shape, tmp_path):
    """Sums of some 1e4 products of unit normals: 1e-13 in FP64, 1e-5 with FP32
    and BF16x3 operands, relative to the norm."""
    args, x, ref = problem
    p = pl.PREC_NAMES[prec]
    ctx = pl.Context(0)
    if shape is not None:
        pl.set_autotune(ctx, 1)
        pl.Heff(ctx, *args, p).free()                       # creates this operator's entry
        f = tmp_path / "plans.tsv"
        pl.autotune_export(str(f))
        keys = [r.split("\t")[0] for r in f.read_text().splitlines() if r]
        f.write_text("".join("%s\t%d\t%d\t%d\n" % (k, shape, shape, 2) for k in keys if k.split("|")[1] == str(p)))
        pl.autotune_import(str(f))
    op = pl.Heff(ctx, *args, p)
    info = op.info()
    assert info["n_T1"] * (8 if prec == "f64" else 4) >= 32 << 20
    y = dev(np.full(len(ref), np.nan))
    op.apply(x, y)
    got = host(y)
    op.free()
    ctx.close()
    assert np.all(np.isfinite(got))
    tol = 1e-13 if prec == "f64" else 1e-5
    assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)
