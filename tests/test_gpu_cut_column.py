"""The truncated beamlets' column form at the edges of its levels and tiles.

Degrees and rows per column follow from how fast erfc's argument varies over
the plane, so the planes below go from a fraction of a waist per column to
several, ragged against its 64 x 128, 64 x 64 and 64 x 32 pixel tiles, with deep cuts,
a dark beamlet and an asymmetric edge set; the pixel-by-pixel form (variant 1)
is the reference beside the oracle.

Tolerances: the truncated Taylor sums leave 2^-25 (mixed) and 2^-50 (FP64) of
a term, the rest is the direct form's rounding: 1e-6 and 1e-12 of the field.
"""
import numpy as np
import pytest

import oracle
import paper_2404_12454_amd as gbd
from paper_2404_12454_amd import scenes
from gbd_testutil import ensure_library, rel_l2

pytestmark = pytest.mark.gpu

TOL = {gbd.GBD_FP64: 1e-12, gbd.GBD_MIXED: 1e-6}


def scene(across, nx, ny, span, deep):
    sc = scenes.truncated_airy_scene(across, npix=nx, npix_y=ny, half_span_lamF=span, z0=1e-4 * deep)
    rng = np.random.default_rng(across + nx)
    cut = np.flatnonzero(np.any(sc.edge != 0, axis=1))
    if deep:
        pick = rng.choice(cut, size=len(cut) // 2, replace=False)
        sc.edge[pick, 2] += rng.uniform(-3.5, 3.5, len(pick)) * sc.w0[0]
    sc.amp[cut[0]] = 0.0
    return sc


@pytest.mark.parametrize("precision", [gbd.GBD_FP64, gbd.GBD_MIXED])
@pytest.mark.parametrize("across,nx,ny,span", [
    (60, 65, 33, 1.0), (40, 64, 64, 4.0), (24, 63, 65, 4.0), (24, 100, 31, 4.0), (16, 70, 24, 8.0), (10, 33, 17, 9.0),
    (30, 1, 40, 3.0), (30, 130, 1, 3.0), (150, 66, 70, 0.8), (140, 65, 129, 1.5)])
@pytest.mark.parametrize("deep", [0, 1])
def test_column_form_matches_oracle_and_direct(across, nx, ny, span, precision, deep):
    ensure_library()
    ctx = gbd.Context(0)
    sc = scene(across, nx, ny, span, deep)
    b, p = gbd.beamlets_from_scene(ctx, sc), gbd.plane_from_scene(ctx, sc)
    ref = oracle.eval_field(sc)
    got = [gbd.gbd_eval(ctx, b, p, precision, opts=o).cpu().numpy().astype(np.complex128)
           for o in (None, dict(variant=1))]
    err = [rel_l2(e, ref) for e in got]
    print(f"{across} across {nx}x{ny} span {span} deep {deep} precision {precision}: {err}", flush=True)
    assert err[0] < TOL[precision] and err[1] < TOL[precision]
