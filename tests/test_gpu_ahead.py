"""gbd_eval launches its evaluation ahead of the setup's status with the route
of the call before: a context that alternates between inputs of different
routes must give each field as a fresh context does, bit for bit."""
import numpy as np
import pytest

import paper_2404_12454_amd as gbd
from paper_2404_12454_amd import scenes
from gbd_testutil import ensure_library

pytestmark = pytest.mark.gpu


def zernike(lens):
    sc = scenes.zernike_scene(7, n_across=70, npix=130, half_span=30e-6)
    m = np.eye(4)
    m[2, 1] = m[3, 0] = lens
    sc.abcd = np.ascontiguousarray((sc.abcd.reshape(-1, 4, 4) @ m).reshape(-1, 16))
    return sc


def rim(waist):
    sc = scenes.truncated_airy_scene(40, npix=96, half_span_lamF=3.0)
    sc.w0 = waist * sc.w0
    return sc


def grid(jitter):
    sc = scenes.airy_scene(24, npix=96, npix_y=80)
    sc.r1 = sc.r1 + np.random.default_rng(2).uniform(-1, 1, sc.r1.shape) * jitter
    return sc


@pytest.mark.parametrize("precision", [gbd.GBD_FP64, gbd.GBD_MIXED])
@pytest.mark.parametrize("make,values", [(zernike, (0.0, 0.05, 0.5, 5.0)), (rim, (1.0, 4.0, 12.0)), (grid, (0.0, 1e-5))])
def test_alternating_inputs_equal_fresh_contexts(make, values, precision):
    import torch
    ensure_library()
    scs = [make(v) for v in values]

    def handles(ctx):
        return [(gbd.beamlets_from_scene(ctx, s), gbd.plane_from_scene(ctx, s)) for s in scs]

    fresh = []
    for i in range(len(scs)):
        ctx = gbd.Context(0)
        b, p = handles(ctx)[i]
        fresh.append(gbd.gbd_eval(ctx, b, p, precision).cpu())
    ctx = gbd.Context(0)
    hs = handles(ctx)
    order = list(range(len(scs))) * 2 + list(range(len(scs)))[::-1]
    got = [(i, gbd.gbd_eval(ctx, *hs[i], precision)) for i in order]
    torch.cuda.synchronize()
    for i, e in got:
        assert torch.equal(torch.view_as_real(e.cpu()), torch.view_as_real(fresh[i])), i
