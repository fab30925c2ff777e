"""One Davidson step on short vectors in one workgroup (launch_dav_step) against
the passes that larger vectors take, on the same basis, products, projected
matrix and diagonal: the library states that both give the same bits.  Called
through the library's own launch functions, at the sizes where the elements a
thread holds change (1, 2, 4), ragged and whole, for the smallest and largest
subspaces of both widths of the passes."""
from ctypes import POINTER, c_bool, c_double, c_int, c_int64, c_void_p

import numpy as np
import pytest

from helpers import pl, dev, host

pytestmark = pytest.mark.gpu
BLOCKS, LD = 1024, 16
PD, STREAM = POINTER(c_double), c_void_p
# the functions of csrc/kernels.hpp, by their linker names
SIGNATURES = {
    "_ZN5pdmrg15launch_dav_stepEPKdS1_liPdibS1_S2_S2_S2_S2_P12ihipStream_t":
        [PD, PD, c_int64, c_int, PD, c_int, c_bool, PD, PD, PD, PD, PD, STREAM],
    "_ZN5pdmrg19launch_dav_ext_gramEPKdS1_lilPdiP12ihipStream_t": [PD, PD, c_int64, c_int, c_int64, PD, c_int, STREAM],
    "_ZN5pdmrg22launch_reduce_partialsEPKdiiPdiP12ihipStream_t": [PD, c_int, c_int, PD, c_int, STREAM],
    "_ZN5pdmrg20launch_dav_g_scatterEPdiiPKdbP12ihipStream_t": [PD, c_int, c_int, PD, c_bool, STREAM],
    "_ZN5pdmrg16launch_small_eigEPKdiiPdS2_P12ihipStream_t": [PD, c_int, c_int, PD, PD, STREAM],
    "_ZN5pdmrg15launch_dav_ritzEPKdS1_liS1_S1_S1_PdS2_S2_S2_lS2_iP12ihipStream_t":
        [PD, PD, c_int64, c_int, PD, PD, PD, PD, PD, PD, PD, c_int64, PD, c_int, STREAM],
    "_ZN5pdmrg18launch_dav_sub_dotEPKdliS1_PdlbS2_iP12ihipStream_t":
        [PD, c_int64, c_int, PD, PD, c_int64, c_bool, PD, c_int, STREAM],
}


def _call(name, *args):
    key, = [k for k in SIGNATURES if k.split("launch_", 1)[1].startswith(name + "E")]
    f = getattr(pl.lib(), key)
    f.argtypes, f.restype = SIGNATURES[key], None
    f(*args, None)


def _p(t, at=0):
    import ctypes
    return ctypes.cast(c_void_p(t.data_ptr() + 8 * at), PD)


def _problem(n, k, seed):
    """Basis of k vectors (orthonormal where n allows), products, the projected matrix without its last row and
    column, a diagonal with an entry the preconditioner has to guard."""
    rng = np.random.default_rng(seed)
    V = rng.standard_normal((k, n))
    if n >= k:
        V = np.linalg.qr(V.T)[0].T
    HV = rng.standard_normal((k, n)) / np.sqrt(n)
    G = np.zeros((LD, LD))
    G[:k - 1, :k - 1] = 0.5 * (V[:k - 1] @ HV[:k - 1].T + HV[:k - 1] @ V[:k - 1].T)
    return dev(V), dev(HV), dev(G), dev(rng.standard_normal(n) + 0.5)


@pytest.mark.parametrize("exact", [False, True])
@pytest.mark.parametrize("k", [1, 2, 8, 9, 16])
@pytest.mark.parametrize("n", [1, 7, 1000, 1024, 1025, 1999, 2048, 2049, 3073, 4095, 4096])
def test_step_has_the_bits_of_the_passes(n, k, exact):
    import torch
    V, HV, G, diag = _problem(n, k, 100 * n + k)
    new = lambda m: torch.full((m,), float("nan"), dtype=torch.float64, device="cuda")
    G1, G2 = G.clone(), G.clone()
    one = [new(n), new(n), new(n), new(8)]                  # x, hx, t, scalars
    _call("dav_step", _p(V), _p(HV), n, k, _p(G1), LD, exact, _p(diag), *[_p(v) for v in one])

    x, hx, r, t, scal, c, dots, partial = new(n), new(n), new(n), new(n), new(64), new(LD), new(64), new(BLOCKS * 64)
    width = pl.lib()["_ZN5pdmrg18dav_ext_gram_widthEi"](k - 1)
    _call("dav_ext_gram", _p(V), _p(HV), n, k - 1, n, _p(partial), BLOCKS)
    _call("reduce_partials", _p(partial), BLOCKS, 2 * width + 1, _p(dots), 1)
    _call("dav_g_scatter", _p(G2), LD, k - 1, _p(dots), exact)
    _call("small_eig", _p(G2), k, LD, _p(scal), _p(c))
    _call("dav_ritz", _p(V), _p(HV), n, k, _p(c), _p(scal), _p(diag), _p(x), _p(hx), _p(r), _p(t), n, _p(partial), BLOCKS)
    _call("reduce_partials", _p(partial), BLOCKS, k + 1, _p(scal, 1), 1)
    _call("dav_sub_dot", _p(V), n, k, _p(scal, 2), _p(t), n, True, _p(partial), BLOCKS)
    _call("reduce_partials", _p(partial), BLOCKS, k, _p(dots), 1)
    _call("dav_sub_dot", _p(V), n, k, _p(dots), _p(t), n, False, _p(partial), BLOCKS)
    _call("reduce_partials", _p(partial), BLOCKS, 1, _p(scal, 2), 1)
    torch.cuda.synchronize()

    assert np.all(np.isfinite(host(scal)[:3])) and np.all(np.isfinite(host(t)))
    assert np.array_equal(host(G1), host(G2))
    for a, b in zip(one, (x, hx, t, scal)):
        m = min(len(a), 3) if b is scal else n
        assert np.array_equal(host(a)[:m], host(b)[:m])
    # and t is orthogonal to the basis
    if n > 2 * k:
        assert np.max(np.abs(host(V) @ host(t))) <= 1e-12 * max(1.0, np.linalg.norm(host(t)))
