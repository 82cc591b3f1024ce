"""Automatic segment counts, lowered to a whole number of workgroups per CU
where a few more would cost a round of their own: grids whose tile counts do
and do not divide the CUs, against the FP64 oracle at the forms' tolerances,
and the count itself (not the first workgroups of another round)."""
import numpy as np
import pytest

import oracle
import paper_2404_12454_amd as gbd
from paper_2404_12454_amd import scenes
from gbd_testutil import ensure_library, rel_l2

pytestmark = pytest.mark.gpu


def jittered(nx, ny):
    sc = scenes.airy_scene(50, npix=nx, npix_y=ny)
    sc.r1 = sc.r1 + np.random.default_rng(2).uniform(-1, 1, sc.r1.shape) * 1e-6
    return sc


def aberrated(nx, ny):
    sc = scenes.zernike_scene(7, n_across=30, npix=nx, half_span=0.1e-6 * nx)
    sc.plane.ny = ny
    return sc


def rim(nx, ny):
    return scenes.truncated_airy_scene(40, npix=nx, npix_y=ny, half_span_lamF=6.0)


@pytest.mark.parametrize("nx,ny", [(300, 257), (256, 256), (409, 275), (130, 65), (17, 700)])
@pytest.mark.parametrize("make", [jittered, aberrated, rim])
@pytest.mark.parametrize("precision,tol", [(gbd.GBD_FP64, 1e-9), (gbd.GBD_MIXED, 1e-6)])
def test_automatic_segments(make, nx, ny, precision, tol):
    import torch
    ensure_library()
    sc = make(nx, ny)
    ctx = gbd.Context(0)
    plan = gbd.Plan(ctx, sc.n).setup(gbd.beamlets_from_scene(ctx, sc), gbd.plane_from_scene(ctx, sc))
    E = plan.eval(precision).cpu()
    assert rel_l2(E.numpy(), oracle.eval_field(sc)) <= tol
    back = plan.eval(precision, opts=plan.shape(precision)).cpu()  # the reported shape gives the same field
    assert torch.equal(torch.view_as_real(back), torch.view_as_real(E))


@pytest.mark.parametrize("make,precision,tile", [(jittered, gbd.GBD_FP64, (128, 128)), (jittered, gbd.GBD_MIXED, (256, 128)),
                                                 (aberrated, gbd.GBD_FP64, (64, 128))])
def test_no_few_workgroups_over_a_round(make, precision, tile):
    import torch
    ensure_library()
    nx, ny = 300, 257
    sc = make(nx, ny)
    ctx = gbd.Context(0)
    plan = gbd.Plan(ctx, sc.n).setup(gbd.beamlets_from_scene(ctx, sc), gbd.plane_from_scene(ctx, sc))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    work = plan.shape(precision)["segments"] * -(-nx // tile[0]) * -(-ny // tile[1])
    assert work % cus == 0 or work % cus > cus // 16 or work < cus
