"""The one-term blocks that stage 1 of a large H_eff writes into T2 have the bits
that the W stage gives them: an operator with T1 past 32 MB, whose right bond is
that of a small one padded with states that nothing couples to, gives the small
one's product bit for bit under the same shape and an unsplit K (the padding adds
zeros to the sums, in whole K steps).  The shapes are those asked for."""
import numpy as np
import pytest

from helpers import pl, synth, blocks_to_flat, flat_to_blocks, dev, host
from oracle import models, mpo as M

pytestmark = pytest.mark.gpu
PQ = (-1, 1)
SITE = 5
BL = {-3: 33, -1: 160, 1: 151, 3: 20}
SMALL = {-3: 32, -1: 64, 1: 32, 3: 64}
PAD = 832                                  # a multiple of every K step
NAMES = ["64x64", "128x32", "32x128", "128x128", "64x64k16", "128x32k16", "64x64k8", "128x32k8", "128x32dma",
         "64x64dma", "32x128dma", "64x64reg", "128x64reg", "64x128reg", "128x128reg", "64x64quad", "128x64quad",
         "64x64quad32", "128x64quad32"]


def _pad(b, rows, cols):
    out = np.zeros((rows, cols))
    out[:b.shape[0], :b.shape[1]] = b
    return out


@pytest.fixture(scope="module")
def problems():
    """(operator arguments, x, table of x) of the small and the padded bond."""
    import torch
    assert torch.cuda.is_available()
    mpo = M.build_mpo(models.heisenberg_terms(models.square_cylinder_bonds(3, 4)), 12, models.OPS, PQ)
    rng = np.random.default_rng(2)
    W1, W2 = (np.array(mpo.W[i], dtype=float) for i in (SITE, SITE + 1))
    W1 *= np.where(W1 == 1.0, 1.0, rng.uniform(0.5, 2.0, W1.shape))
    dl, dm, dr = mpo.deltas[SITE], mpo.deltas[SITE + 1], mpo.deltas[SITE + 2]
    L, R = synth.random_env_blocks(BL, dl, rng), synth.random_env_blocks(SMALL, dr, rng)
    psi = synth.random_two_site_blocks(BL, SMALL, PQ, rng)
    out = []
    for br in (SMALL, {q: n + PAD for q, n in SMALL.items()}):
        Rb = {(q, w): _pad(b, br[q], br[q - int(dr[w])]) for (q, w), b in R.items()}
        xb = {(q, s, t): _pad(b, b.shape[0], br[q + PQ[s] + PQ[t]]) for (q, s, t), b in psi.items()}
        B1, B2, P = pl.Bond(BL), pl.Bond(br), pl.Phys(PQ)
        tx, nx = pl.layout(pl.TWO_SITE, B1, B2, P)
        tl, nl = pl.layout(pl.ENV_L, B1, deltas=dl)
        tr, nr = pl.layout(pl.ENV_R, B2, deltas=dr)
        args = (B1, B2, P, pl.MpoSite(W1, dl, dm), pl.MpoSite(W2, dm, dr),
                dev(blocks_to_flat(L, tl, nl, pl.ENV_L)), dev(blocks_to_flat(Rb, tr, nr, pl.ENV_R)))
        out.append((args, dev(blocks_to_flat(xb, tx, nx, pl.TWO_SITE)), tx))
    return out


@pytest.mark.parametrize("prec,shape", [("f64", s) for s in range(15)] +
                         [("f32", s) for s in list(range(11)) + [15, 16, 17, 18]] +
                         [("bf16x3", s) for s in (8, 9, 10, 15, 16, 17, 18)])
def test_direct_blocks_keep_the_bits(problems, prec, shape, tmp_path):
    p = pl.PREC_NAMES[prec]
    ctx = pl.Context(0)
    pl.set_autotune(ctx, 1)
    f = tmp_path / "plans.tsv"
    for args, _, _ in problems:
        pl.Heff(ctx, *args, p).free()                       # creates this operator's entry
    pl.autotune_export(str(f))
    keys = [r.split("\t")[0] for r in f.read_text().splitlines() if r]
    keys = [k for k in keys if k.split("|")[1] == str(p)]
    assert len(keys) >= 2
    f.write_text("".join("%s\t%d\t%d\t1\n" % (k, shape, shape) for k in keys))
    pl.autotune_import(str(f))
    got, t1 = [], []
    for args, x, table in problems:
        op = pl.Heff(ctx, *args, p)
        info = op.info()
        assert info["shape_Lpsi"] == info["shape_R"] == NAMES[shape]
        t1.append(info["n_T1"] * (8 if prec == "f64" else 4))
        y = dev(np.full(x.numel(), np.nan))
        op.apply(x, y)
        got.append(flat_to_blocks(host(y), table, pl.TWO_SITE))
        op.free()
    ctx.close()
    assert t1[0] < 32 << 20 <= t1[1]
    for k, b in got[0].items():
        assert np.all(np.isfinite(b)) and np.linalg.norm(b) > 0.0
        assert np.array_equal(got[1][k][:, :b.shape[1]], b), k
        assert not np.any(got[1][k][:, b.shape[1]:])
