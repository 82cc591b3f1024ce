"""Beamlet handles' uploads: arrays in the caller's order are copied whole,
and every element is checked.

Each optional array given or left out, one or many waists and matrices, must
give the field of the same handle stored in another order (a truncating edge
moved to the front makes the packing go beamlet by beamlet); a fault in the
last element of any array is refused.
"""
import numpy as np
import pytest

import paper_2404_12454_amd as gbd
from paper_2404_12454_amd import scenes
from gbd_testutil import ensure_library, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    ensure_library()
    return gbd.Context(0)


def arrays(sc, many):
    n = sc.n
    rng = np.random.default_rng(4)
    return dict(r1=sc.r1.copy(), th1=rng.uniform(-1e-6, 1e-6, (n, 2)), w0=np.full(n if many else 1, sc.w0[0]),
                amp=np.stack([np.full(n, 0.7), rng.uniform(-1, 1, n)], 1), path=rng.uniform(0, 1e-7, n),
                abcd=np.tile(sc.abcd.reshape(-1, 16), (n if many else 1, 1)))


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("absent", [(), ("th1",), ("amp",), ("path",), ("th1", "amp", "path")])
def test_whole_array_upload_is_the_element_wise_one(ctx, many, absent):
    sc = scenes.airy_scene(13, npix=40)
    a = arrays(sc, many)
    for k in absent:
        a[k] = None
    p = gbd.plane_from_scene(ctx, sc)
    n = sc.n
    args = [a[k] for k in ("r1", "th1", "w0", "amp", "path", "abcd")]
    whole = gbd.gbd_eval(ctx, raw(ctx, sc, args, None), p, gbd.GBD_FP64)
    # the first beamlet cut by an edge far outside its waist: whole, but stored last
    edge = np.zeros((n, 3))
    edge[0] = [1.0, 0.0, 1.0]
    packed = gbd.gbd_eval(ctx, raw(ctx, sc, args, edge), p, gbd.GBD_FP64)
    assert rel_l2(packed.cpu().numpy(), whole.cpu().numpy()) < 1e-12


def raw(ctx, sc, args, edge):
    import ctypes
    lib = gbd.load_library()
    arr = [None if x is None else np.ascontiguousarray(x, np.float64) for x in args]
    r1, th1, w0, amp, path, abcd = arr
    ptr = [None if x is None else x.ctypes.data_as(ctypes.c_void_p) for x in arr]
    h = ctypes.c_void_p()
    head = (ctx.handle, ctypes.byref(h), sc.n, sc.lam, sc.l0, ptr[0], ptr[1], ptr[2], w0.size, ptr[3], ptr[4], ptr[5],
            abcd.size // 16)
    rc = (lib.gbd_beamlets(*head) if edge is None else
          lib.gbd_beamlets_truncated(*head, edge.ctypes.data_as(ctypes.c_void_p)))
    if rc:
        raise gbd.GbdError(rc, "refused")
    return gbd.Beamlets(h, sc.n)


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("name", ["r1", "th1", "w0", "amp", "path", "abcd"])
def test_last_element_is_checked(ctx, name, value):
    sc = scenes.airy_scene(13, npix=8)
    a = arrays(sc, True)
    a[name].reshape(-1)[-1] = value
    with pytest.raises(gbd.GbdError):
        gbd.gbd_beamlets(ctx, sc.n, sc.lam, sc.l0, *(a[k] for k in ("r1", "th1", "w0", "amp", "path", "abcd")))


@pytest.mark.parametrize("entry", range(16))
@pytest.mark.parametrize("traced", [False, True])
def test_last_matrix_is_checked(ctx, entry, traced):
    """Every entry of a lens-and-distance matrix takes part in M^T J M = J
    (with equal focal lengths D = 0, so A's entries only against B's and C's)."""
    sc = scenes.airy_scene(13, npix=8)
    a = arrays(sc, True)
    m = np.eye(4)
    m[:2, 2:] = 0.3 * np.eye(2) + 0.01
    m[2:, :2] = -0.2 * np.eye(2)
    m[:2, :2] += m[:2, 2:] @ m[2:, :2]
    a["abcd"][:] = m.reshape(-1)
    names = ("r1", "th1", "w0", "amp", "path", "abcd")

    def make():
        if traced:
            return gbd.gbd_beamlets_traced(ctx, sc.n, sc.lam, sc.l0, *(a[k] for k in names), np.zeros((sc.n, 5)))
        return gbd.gbd_beamlets(ctx, sc.n, sc.lam, sc.l0, *(a[k] for k in names))

    make()
    a["abcd"][-1, entry] += 1e-3
    with pytest.raises(gbd.GbdError):
        make()
