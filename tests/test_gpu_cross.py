"""The matrix form for weak cross terms (tilted, aberrated planes) against the
FP64 oracle at 1e-6 relative L2, twice the rotor form's error: both levels of
its series, grids at the edges of its 128 x 128 tiles and 16 x 16 blocks,
beamlet counts at the edges of its passes, and what it leaves to the rotor
form (one segment, other launch shapes, stronger cross terms)."""
import numpy as np
import pytest

import oracle
import paper_2404_12454_amd as gbd
from paper_2404_12454_amd import scenes
from gbd_testutil import ensure_library, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    ensure_library()
    return gbd.Context(0)


def scene(across, nx, ny, pitch, seed=11):
    s = scenes.zernike_scene(seed, n_across=across, npix=nx, half_span=0.5 * nx * pitch)
    s.plane.ny = ny
    return s


def plan_of(ctx, sc):
    return gbd.Plan(ctx, sc.n).setup(gbd.beamlets_from_scene(ctx, sc), gbd.plane_from_scene(ctx, sc))


# pitches 0.05 and 0.2 um: 1.0e-3 and 1.6e-2 bound the corner's cross term at
# these beamlet counts, one level each
@pytest.mark.parametrize("pitch", [0.05e-6, 0.15e-6])
@pytest.mark.parametrize("across,nx,ny,seg", [(40, 127, 65, 0), (40, 128, 128, 2), (48, 129, 17, 3), (40, 300, 140, 5),
                                              (64, 16, 129, 40), (40, 257, 255, 0)])
def test_cross_form_ragged(ctx, pitch, across, nx, ny, seg):
    import torch
    sc = scene(across, nx, ny, pitch)
    plan = plan_of(ctx, sc)
    o = dict(segments=seg) if seg else None
    shape = plan.shape(gbd.GBD_MIXED, o)
    assert shape["variant"] == 3 and (shape["rows_per_lane"], shape["waves"]) == (32, 4) and shape["segments"] >= 2
    E = plan.eval(gbd.GBD_MIXED, opts=o).cpu()
    assert rel_l2(E.numpy(), oracle.eval_field(sc)) <= 1e-6
    back = plan.eval(gbd.GBD_MIXED, opts=shape).cpu()  # the reported shape gives the same field
    assert torch.equal(back.view(torch.float32), E.view(torch.float32))


@pytest.mark.parametrize("n,seg", [(130, 2), (131, 9), (255, 4), (256, 8), (257, 16), (1000, 7)])
def test_cross_form_short_and_ragged_segments(ctx, n, seg):
    full = scene(40, 200, 180, 0.1e-6)
    keep = np.zeros(full.n, bool)
    keep[np.random.default_rng(n).choice(full.n, n, replace=False)] = True
    sc = oracle._subset(full, keep)
    sc.amp = sc.amp * (10.0 ** np.random.default_rng(1).uniform(-9, 3, n))[:, None]
    E = plan_of(ctx, sc).eval(gbd.GBD_MIXED, opts=dict(segments=seg)).cpu().numpy()
    assert rel_l2(E, oracle.eval_field(sc)) <= 1e-6


def test_cross_form_leaves_one_segment_and_other_shapes_to_the_rotor_form(ctx):
    """One segment is the batched sweep's arithmetic (bit for bit); other rows and wavefronts the rotor's."""
    import torch
    sc = scene(40, 160, 144, 0.1e-6)
    ref = oracle.eval_field(sc)
    b, p = gbd.beamlets_from_scene(ctx, sc), gbd.plane_from_scene(ctx, sc)
    plan = gbd.Plan(ctx, sc.n).setup(b, p)
    for o in (dict(segments=1), dict(rows_per_lane=16, waves=4), dict(rows_per_lane=32, waves=2), dict(variant=1)):
        assert rel_l2(plan.eval(gbd.GBD_MIXED, opts=o).cpu().numpy(), ref) <= 1e-6
    _, fields = gbd.gbd_eval_batch(ctx, [b], [p], fields=True)
    E = plan.eval(gbd.GBD_MIXED, opts=dict(segments=1, variant=3, rows_per_lane=32, waves=4)).cpu()
    assert torch.equal(fields[0].cpu().view(torch.float32), E.view(torch.float32))


def test_cross_form_from_call_to_call(ctx):
    """gbd_eval's launch ahead over planes of level 1, level 2, none, and no cross terms at all."""
    import torch
    ss = [scene(40, 160, 144, h) for h in (0.05e-6, 0.15e-6, 1.0e-6)] + [scenes.airy_scene(24, npix=100)]
    hs = [(gbd.beamlets_from_scene(ctx, s), gbd.plane_from_scene(ctx, s)) for s in ss]
    want = []
    for s in ss:
        fresh = gbd.Context(0)
        want.append(gbd.gbd_eval(fresh, gbd.beamlets_from_scene(fresh, s), gbd.plane_from_scene(fresh, s)).cpu())
        assert rel_l2(want[-1].numpy(), oracle.eval_field(s)) <= 1e-6
    for i in (0, 0, 1, 1, 2, 2, 0, 2, 1, 0, 3, 3, 0, 1, 3, 2):
        E = gbd.gbd_eval(ctx, *hs[i]).cpu()
        assert torch.equal(E.view(torch.float32), want[i].view(torch.float32)), i


@pytest.mark.parametrize("pitch", [0.05e-6, 0.15e-6])
@pytest.mark.parametrize("weak", [1.0, 1e-3, 1e-9])
def test_cross_form_masked_beamlets(ctx, pitch, weak):
    """Beamlets of zero amplitude in fields down to 1e-9, both levels: their factors are zero, not infinite."""
    sc = scene(40, 200, 180, pitch)
    sc.amp = weak * sc.amp
    sc.amp[::5] = 0.0
    sc.amp[100:300] = 0.0
    E = plan_of(ctx, sc).eval(gbd.GBD_MIXED, opts=dict(segments=3)).cpu().numpy()
    assert rel_l2(E, oracle.eval_field(sc)) <= 1e-6
    assert rel_l2(gbd.gbd_eval(ctx, gbd.beamlets_from_scene(ctx, sc), gbd.plane_from_scene(ctx, sc)).cpu().numpy(),
                  oracle.eval_field(sc)) <= 1e-6


def test_cross_form_keeps_its_sums_short(ctx):
    """100,668 beamlets: the plain FP32 sums stay short enough for the rotor form's error, whether the segment count
    is automatic, given, or lowered to the static buffer's 4; too few segments are the rotor form's."""
    import torch
    sc = scene(358, 1024, 1024, 0.25e-6)
    plan = plan_of(ctx, sc)
    ref = plan.eval(gbd.GBD_FP64).cpu().numpy()
    assert plan.shape(gbd.GBD_MIXED)["segments"] * 656 >= sc.n
    fields = {k: plan.eval(gbd.GBD_MIXED, opts=dict(segments=k) if k else None).cpu() for k in (0, 4, 7, 16, 160)}
    fields["static"] = plan.eval_noalloc(gbd.GBD_MIXED).cpu()
    err = {k: rel_l2(E.numpy(), ref) for k, E in fields.items()}
    print(err, flush=True)
    assert max(err.values()) <= 1e-6
    assert torch.equal(fields["static"].view(torch.float32), fields[4].view(torch.float32))


def test_low_planes_keep_the_rotor_forms_rows(ctx):
    """Fewer than 128 rows: the rotor form's 16 rows where the cross form does not run (one segment, or a static
    buffer too small for its sums)."""
    import torch
    sc = scene(100, 2000, 120, 0.1e-6)
    plan = plan_of(ctx, sc)
    assert plan.shape(gbd.GBD_MIXED, dict(segments=1))["rows_per_lane"] == 16
    ref = plan.eval(gbd.GBD_FP64).cpu().numpy()
    room = (64 << 20) // (2000 * 120 * 16)
    E = plan.eval_noalloc(gbd.GBD_MIXED).cpu()
    assert rel_l2(E.numpy(), ref) <= 4e-7  # 16 rows; 32 rows 4.5e-7 and more
    rotor = plan.eval(gbd.GBD_MIXED, opts=dict(rows_per_lane=16, waves=4, segments=room)).cpu()
    assert torch.equal(E.view(torch.float32), rotor.view(torch.float32))
    assert rel_l2(plan.eval(gbd.GBD_MIXED).cpu().numpy(), ref) <= 4e-7


def test_cross_form_is_no_less_exact_than_the_rotor_form(ctx):
    """15,856 beamlets on 323 x 433 pixels, where the automatic count once left 755 to a sum: against the rotor form's
    32 rows at the same count."""
    sc = scenes.zernike_scene(808388750, n_across=142, npix=323, half_span=7.176e-5, tilt_deg=0.0, defocus=5.0705e-5)
    sc.plane.ny = 433
    plan = plan_of(ctx, sc)
    ref = plan.eval(gbd.GBD_FP64).cpu().numpy()
    k = plan.shape(gbd.GBD_MIXED)["segments"]
    cross = rel_l2(plan.eval(gbd.GBD_MIXED).cpu().numpy(), ref)
    rotor = rel_l2(plan.eval(gbd.GBD_MIXED, opts=dict(rows_per_lane=32, waves=2, segments=k)).cpu().numpy(), ref)
    print(f"{k} segments: cross {cross:.2e}, rotor {rotor:.2e}", flush=True)
    assert cross <= rotor
