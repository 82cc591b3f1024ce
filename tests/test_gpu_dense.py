"""The separable form by beamlets (dense), which beamlets stored in no order
and captured evaluations take, against the FP64 oracle where grids stored row
by row go by rows instead: ragged grids and segments, amplitude ranges, the
cap on the FP32 sums, automatic counts.  Tolerances as everywhere (relative L2
1e-12 FP64, 1e-5 mixed)."""
import numpy as np
import pytest

import oracle
import paper_2404_12454_amd as gbd
from paper_2404_12454_amd import scenes
from gbd_testutil import ensure_library, rel_l2

pytestmark = pytest.mark.gpu

TOL = {gbd.GBD_FP64: 1e-12, gbd.GBD_MIXED: 1e-5}
BOTH = [gbd.GBD_FP64, gbd.GBD_MIXED]


@pytest.fixture(scope="module")
def ctx():
    ensure_library()
    return gbd.Context(0)


def permuted(sc, seed=1):
    """The same beamlets in no order: no runs of one row."""
    p = np.random.default_rng(seed).permutation(sc.n)
    out = scenes.Scene(sc.lam, sc.l0, sc.r1[p], sc.th1[p], sc.w0[p], sc.amp[p], sc.path[p], sc.abcd, sc.plane)
    if sc.order is not None:
        out.order = sc.order[p]
    return out


def plan_of(ctx, sc):
    return gbd.Plan(ctx, sc.n).setup(gbd.beamlets_from_scene(ctx, sc), gbd.plane_from_scene(ctx, sc))


@pytest.mark.parametrize("precision", BOTH)
@pytest.mark.parametrize("make", [scenes.airy_scene, scenes.hermite_scene])
@pytest.mark.parametrize("nx,ny,seg", [(70, 45, 1), (70, 45, 3), (129, 200, 0), (1, 1, 1), (65, 1, 2), (1, 70, 0),
                                       (300, 97, 5)])
def test_ragged_grids(ctx, make, nx, ny, seg, precision):
    sc = permuted(make(21, npix=nx, npix_y=ny, half_span_lamF=8.0, z0=30e-6))
    plan = plan_of(ctx, sc)
    assert plan.shape(precision, dict(segments=seg))["variant"] == 4
    assert rel_l2(plan.eval(precision, opts=dict(segments=seg)).cpu().numpy(), oracle.eval_field(sc)) <= TOL[precision]


@pytest.mark.parametrize("scale,spread", [(1e12, 1.0), (1e-12, 1.0), (1.0, 1e-9), (1e6, 1e-14)])
def test_halves_across_amplitude_ranges(ctx, scale, spread):
    """Uniform amplitudes far from 1, and half of the beamlets weaker by `spread`, on a defocused grid."""
    sc = scenes.airy_scene(24, npix=96, npix_y=80, half_span_lamF=8.0, z0=200e-6)
    sc.amp = sc.amp * scale
    sc.amp[::2] *= spread
    sc = permuted(sc)
    ref = oracle.eval_field(sc)
    plan = plan_of(ctx, sc)
    for variant in (4, 5):
        assert rel_l2(plan.eval(gbd.GBD_MIXED, opts=dict(variant=variant)).cpu().numpy(), ref) <= TOL[gbd.GBD_MIXED]


@pytest.mark.parametrize("segments", [1, 5])
def test_explicit_segments_respect_the_fp32_cap(ctx, segments):
    """205,898 beamlets: counts that would leave more than 16,384 to an FP32 sum are raised."""
    sc = permuted(scenes.airy_scene(512, npix=48, npix_y=40, half_span_lamF=6.0))
    plan = plan_of(ctx, sc)
    o = dict(segments=segments)
    assert -(-sc.n // plan.shape(gbd.GBD_MIXED, o)["segments"]) <= 16384
    assert rel_l2(plan.eval(gbd.GBD_MIXED, opts=o).cpu().numpy(), oracle.eval_field(sc)) <= TOL[gbd.GBD_MIXED]


def test_long_automatic_segments_are_split(ctx):
    """823,592 beamlets on 512 x 512 pixels: at most 16,384 to an FP32 sum, sampled pixels."""
    sc = permuted(scenes.airy_scene(1024, npix=512, half_span_lamF=20.0))
    plan = plan_of(ctx, sc)
    assert plan.shape(gbd.GBD_MIXED)["segments"] * 16384 >= sc.n
    E = plan.eval(gbd.GBD_MIXED).cpu().numpy()
    ix, iy = np.random.default_rng(8).integers(0, 512, (2, 60)).astype(np.int32)
    assert rel_l2(E[iy, ix], oracle.eval_field(sc, pixels=(ix, iy))) <= TOL[gbd.GBD_MIXED]


@pytest.mark.parametrize("precision", BOTH)
@pytest.mark.parametrize("nx,ny", [(300, 257), (256, 256), (130, 65)])
def test_automatic_counts(ctx, nx, ny, precision):
    sc = permuted(scenes.airy_scene(50, npix=nx, npix_y=ny))
    assert rel_l2(plan_of(ctx, sc).eval(precision).cpu().numpy(), oracle.eval_field(sc)) <= TOL[precision]
