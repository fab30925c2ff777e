"""Gradient of one MPO tensor where its products change shape: blocks under, at
and over one chunk of 2048 numbers, lists of 1, 4, 5, 64, 65 and 130 channels,
more than 16 blocks on one entry, entries that no block reaches."""
import numpy as np
import pytest

from helpers import pl, synth, blocks_to_flat, dev, host

pytestmark = pytest.mark.gpu
PQ = (-1, 1)

BONDS = {
    "one": ({0: 1}, {-1: 1, 1: 1}),
    "chunk": ({-1: 5, 1: 33}, {-2: 32, 0: 64, 2: 45}),                       # 32 x 64, 45 x 45, 64 x 64 blocks
    "many": ({q: 3 for q in range(-20, 21, 2)}, {q: 2 + abs(q) % 5 for q in range(-21, 22, 2)}),
}


@pytest.mark.parametrize("channels", [1, 4, 5, 64, 65, 130])
@pytest.mark.parametrize("bonds", sorted(BONDS))
def test_gradient_of_wide_mpo_sites(bonds, channels):
    """Sums of at most 1e5 products of unit normals, relative to their norm:
    1e-13."""
    import torch
    assert torch.cuda.is_available()
    bl, br = BONDS[bonds]
    rng = np.random.default_rng(channels)
    d, Dl, Dr = 2, 3, channels
    dl, dr = np.array([0, 2, 0]), np.array([(0, 2, -2)[w % 3] if w % 7 else 0 for w in range(Dr)])
    A = synth.random_site_blocks(bl, br, PQ, rng)
    L, R = synth.random_env_blocks(bl, dl, rng), synth.random_env_blocks(br, dr, rng)
    B1, B2, P = pl.Bond(bl), pl.Bond(br), pl.Phys(PQ)
    ta, na = pl.layout(pl.SITE, B1, B2, P)
    tl, nl = pl.layout(pl.ENV_L, B1, deltas=dl)
    tr, nr = pl.layout(pl.ENV_R, B2, deltas=dr)
    ctx = pl.Context(0)
    W = pl.MpoSite(np.zeros((Dl, d, d, Dr)), dl, dr)
    got = host(pl.grad_site(ctx, B1, B2, P, W, dev(blocks_to_flat(L, tl, nl, pl.ENV_L)),
                            dev(blocks_to_flat(A, ta, na, pl.SITE)), dev(blocks_to_flat(R, tr, nr, pl.ENV_R))))
    ctx.close()
    ref = np.zeros((Dl, d, d, Dr))
    for (qa, s), Aq in A.items():
        for w in range(Dl):
            Lb = L.get((qa, w))
            if Lb is None:
                continue
            for t in range(d):
                At = A.get((qa - int(dl[w]), t))
                if At is None:
                    continue
                Z = Aq.T @ Lb @ At                  # [b][b']
                for w2 in range(Dr):
                    Rb = R.get((qa + PQ[s], w2))
                    if Rb is not None and qa + PQ[s] - int(dr[w2]) == qa - int(dl[w]) + PQ[t]:
                        ref[w, s, t, w2] += np.sum(Z * Rb)
    assert got.shape == ref.shape and np.all(np.isfinite(got))
    assert np.linalg.norm(got - ref) <= 1e-13 * max(np.linalg.norm(ref), 1e-300)
    assert np.array_equal(got == 0.0, ref == 0.0)
