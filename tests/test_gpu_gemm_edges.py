"""H_eff with the register-direct (FP64) and quad (FP32, BF16x3) GEMM shapes at the
edges of their tiles: bonds whose sectors are one row wide, odd, just under, at
and over the 16 / 32 / 64 / 128 boundaries of the wave and workgroup tiles and
of the K steps, forced through imported tuning entries, against the same
contraction on dense NumPy blocks."""
import numpy as np
import pytest

from helpers import pl, synth, blocks_to_flat, dev, host, mpo_site
from oracle import models, dmrg, mpo as M
from oracle.blocks import Bond

pytestmark = pytest.mark.gpu
PQ = (-1, 1)
NAMES = {11: "64x64reg", 12: "128x64reg", 13: "64x128reg", 14: "128x128reg",
         15: "64x64quad", 16: "128x64quad", 17: "64x64quad32", 18: "128x64quad32"}
PLANS = [("f64", s, p) for s in (11, 12, 13, 14) for p in (1, 16)] + \
    [(t, s, p) for t in ("f32", "bf16x3") for s in (15, 16, 17, 18) for p in (1, 8)]
SITE = 5

# (left bond, right bond) of a two-site problem
BONDS = [
    ({-1: 1, 1: 1}, {-1: 1, 1: 1}),
    ({-1: 7, 1: 9}, {-1: 8, 1: 17}),
    ({-1: 31, 1: 33}, {-1: 63, 1: 2}),
    ({-1: 64, 1: 127}, {-1: 129, 1: 31}),
    ({-3: 5, -1: 131, 1: 70}, {-1: 193, 1: 24, 3: 1}),
]


@pytest.fixture(scope="module")
def mpo():
    return M.build_mpo(models.heisenberg_terms(models.square_cylinder_bonds(3, 4)), 12, models.OPS, PQ)


@pytest.mark.parametrize("prec,shape,parts", PLANS)
@pytest.mark.parametrize("case", range(len(BONDS)))
def test_heff_tile_edges(mpo, case, prec, shape, parts, tmp_path):
    """Sums of at most a few thousand terms: 1e-13 relative in FP64, 1e-5 with
    FP32 and BF16x3 operands.  x, the environments and y lie inside buffers of NaN: a value read past an operand
    that reached a product would make the result NaN."""
    import torch
    bl, br = BONDS[case]
    rng = np.random.default_rng(case)
    dl, dr = mpo.deltas[SITE], mpo.deltas[SITE + 2]
    L, R = synth.random_env_blocks(bl, dl, rng), synth.random_env_blocks(br, dr, rng)
    psi = synth.random_two_site_blocks(bl, br, PQ, rng)
    B1, B2, P = pl.Bond(bl), pl.Bond(br), pl.Phys(PQ)
    tx, nx = pl.layout(pl.TWO_SITE, B1, B2, P)
    tl, nl = pl.layout(pl.ENV_L, B1, deltas=dl)
    tr, nr = pl.layout(pl.ENV_R, B2, deltas=dr)
    pool = torch.full((2 * nx + nl + nr + 80,), float("nan"), dtype=torch.float64, device="cuda")
    ends, views = 16, []
    for flat in (blocks_to_flat(psi, tx, nx, pl.TWO_SITE), np.full(nx, np.nan), blocks_to_flat(L, tl, nl, pl.ENV_L),
                 blocks_to_flat(R, tr, nr, pl.ENV_R)):
        views.append(pool[ends:ends + len(flat)])
        views[-1].copy_(dev(flat))
        ends += len(flat) + 16
    x, y, Ld, Rd = views

    ctx = pl.Context(0)
    pl.set_autotune(ctx, 1)
    args = (ctx, B1, B2, P, mpo_site(mpo, SITE), mpo_site(mpo, SITE + 1), Ld, Rd, pl.PREC_NAMES[prec])
    pl.Heff(*args).free()                                   # creates this operator's entry
    f = tmp_path / "plans.tsv"
    pl.autotune_export(str(f))
    keys = [r.split("\t")[0] for r in f.read_text().splitlines() if r]
    f.write_text("".join("%s\t%d\t%d\t%d\n" % (k, shape, shape, parts) for k in keys if k.split("|")[1] == str(pl.PREC_NAMES[prec])))
    pl.autotune_import(str(f))
    op = pl.Heff(*args)
    info = op.info()
    assert info["shape_Lpsi"] == info["shape_R"] == NAMES[shape]
    op.apply(x, y)
    got = host(y)
    op.free()
    ctx.close()
    ref = dmrg.heff_apply(L, R, mpo.W[SITE], mpo.W[SITE + 1], psi, Bond(bl), Bond(br), PQ, dl, dr)
    ref = blocks_to_flat(ref, tx, nx, pl.TWO_SITE)
    assert np.all(np.isfinite(got))
    assert np.linalg.norm(got - ref) <= (1e-13 if prec == "f64" else 1e-5) * np.linalg.norm(ref)
    gap = pool[32 + nx - 16:32 + nx]                        # around y, still untouched
    assert bool(torch.isnan(gap).all()) and bool(torch.isnan(pool[32 + 2 * nx:48 + 2 * nx]).all())
