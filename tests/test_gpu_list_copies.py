"""Work lists on their way to the device: environment updates and gradients of
several bonds, on contexts with streams of their own and from several host
threads at once, keep the bits they have one at a time; pinned and device blocks
outlive neither an error nor the last context."""
import threading

import numpy as np
import pytest

from helpers import pl, synth, blocks_to_flat, dev, mpo_site
from oracle import models, mpo as M

pytestmark = pytest.mark.gpu
PQ = (-1, 1)
SITES = (2, 5, 8)
BONDS = [({-1: 7, 1: 9}, {-2: 3, 0: 15, 2: 1}), ({-1: 31, 1: 33}, {-2: 1, 0: 65, 2: 32}), ({-1: 1, 1: 1}, {0: 1})]


@pytest.fixture(scope="module")
def mpo():
    return M.build_mpo(models.heisenberg_terms(models.square_cylinder_bonds(3, 4)), 12, models.OPS, PQ)


def _problem(mpo, k):
    """Inputs of the one-site problem k, on the device."""
    (bl, br), i = BONDS[k], SITES[k]
    rng = np.random.default_rng(k)
    B1, B2, P = pl.Bond(bl), pl.Bond(br), pl.Phys(PQ)
    ta, na = pl.layout(pl.SITE, B1, B2, P)
    tl, nl = pl.layout(pl.ENV_L, B1, deltas=mpo.deltas[i])
    tr, nr = pl.layout(pl.ENV_R, B2, deltas=mpo.deltas[i + 1])
    to, no = pl.layout(pl.ENV_L, B2, deltas=mpo.deltas[i + 1])
    A = dev(blocks_to_flat(synth.random_site_blocks(bl, br, PQ, rng), ta, na, pl.SITE))
    L = dev(blocks_to_flat(synth.random_env_blocks(bl, mpo.deltas[i], rng), tl, nl, pl.ENV_L))
    R = dev(blocks_to_flat(synth.random_env_blocks(br, mpo.deltas[i + 1], rng), tr, nr, pl.ENV_R))
    return B1, B2, P, mpo_site(mpo, i), L, A, R, no


def _results(ctx, problems, order):
    import torch
    out = {}
    for k in order:
        B1, B2, P, W, L, A, R, no = problems[k]
        e = torch.full((no,), float("nan"), dtype=torch.float64, device="cuda")
        pl.env_update(ctx, 1, B1, B2, P, W, L, A, e)
        out[k] = (e.cpu().numpy(), pl.grad_site(ctx, B1, B2, P, W, L, A, R).cpu().numpy())
    return out


@pytest.mark.parametrize("threads", [1, 3])
def test_lists_of_several_streams_keep_their_bits(mpo, threads):
    import torch
    problems = [_problem(mpo, k) for k in range(len(BONDS))]
    ref_ctx = pl.Context(0)
    ref = _results(ref_ctx, problems, range(len(problems)))
    streams = [torch.cuda.Stream() for _ in range(threads)]
    torch.cuda.synchronize()
    got, fail = [None] * threads, []

    def work(t):
        try:
            with torch.cuda.stream(streams[t]):
                c = pl.Context(0, streams[t])
                order = [(k + t) % len(problems) for k in range(len(problems))] * 8
                got[t] = _results(c, problems, order)
                c.close()
        except Exception as e:              # noqa: BLE001 - reported by the main thread
            fail.append(e)

    pool = [threading.Thread(target=work, args=(t,)) for t in range(threads)]
    for p in pool:
        p.start()
    for p in pool:
        p.join()
    assert not fail, fail
    for g in got:
        for k, (e, grad) in ref.items():
            assert np.array_equal(g[k][0], e) and np.array_equal(g[k][1], grad)
    ref_ctx.close()                         # the last context: the blocks are given back
    again = pl.Context(0)
    out = _results(again, problems, [1])
    assert np.array_equal(out[1][0], ref[1][0])
    again.close()


def test_a_refused_mpo_leaves_the_context_usable(mpo):
    """An MPO entry that breaks charge conservation is found while the first
    product runs: refused, with nothing written, and the next call is right."""
    import torch
    ctx = pl.Context(0)
    problems = [_problem(mpo, k) for k in range(len(BONDS))]
    ref = _results(ctx, problems, [1])
    B1, B2, P, W, L, A, R, no = problems[1]
    i = SITES[1]
    bad = np.array(mpo.W[i], dtype=np.float64)
    w = int(np.flatnonzero(np.asarray(mpo.deltas[i]) == 0)[0])
    w2 = int(np.flatnonzero(np.asarray(mpo.deltas[i + 1]) == 0)[0])
    bad[w, 0, 1, w2] = 1.0
    Wbad = pl.MpoSite(bad, mpo.deltas[i], mpo.deltas[i + 1])
    out = torch.full((no,), 7.0, dtype=torch.float64, device="cuda")
    with pytest.raises(pl.PdmrgError):
        pl.env_update(ctx, 1, B1, B2, P, Wbad, L, A, out)
    torch.cuda.synchronize()
    assert bool((out == 7.0).all())
    again = _results(ctx, problems, [1])
    assert np.array_equal(again[1][0], ref[1][0]) and np.array_equal(again[1][1], ref[1][1])
    ctx.close()
