"""The allocation-free entry point (gbd_plan_eval_noalloc) against
gbd_plan_eval, through the C ABI.

Its segment partial sums live in the library's static per-device buffer,
which keeps the previous call's contents; so every case runs two calls in a
row, the second on a smaller input, and compares each with gbd_plan_eval on
the same plan: bit for bit where the resolved launch shape is the same, and
to the mixed / FP64 tolerances (1e-5 / 1e-12 relative L2) where the static
buffer lowers the automatic segment count.
"""
import numpy as np
import pytest

import oracle
import paper_2404_12454_amd as gbd
from paper_2404_12454_amd import scenes
from gbd_testutil import ensure_library, rel_l2

pytestmark = pytest.mark.gpu

TOL = {gbd.GBD_FP64: 1e-12, gbd.GBD_MIXED: 1e-5}
BOTH = [gbd.GBD_FP64, gbd.GBD_MIXED]
LIMIT = 64 << 20  # GBD_NOALLOC_SCRATCH_BYTES


@pytest.fixture(scope="module")
def ctx():
    ensure_library()
    return gbd.Context(0)


def plan_of(ctx, sc):
    return gbd.Plan(ctx, sc.n).setup(gbd.beamlets_from_scene(ctx, sc), gbd.plane_from_scene(ctx, sc))


def pair(ctx, big, small, precision):
    """Reference fields first, then the allocation-free calls back to back
    (big, then small), then the comparison."""
    import torch
    plans = [plan_of(ctx, big), plan_of(ctx, small)]
    refs = [p.eval(precision) for p in plans]
    got = [p.eval_noalloc(precision) for p in plans]
    torch.cuda.synchronize()
    return plans, [r.cpu() for r in refs], [g.cpu() for g in got]


def bits(t):
    import torch
    return t.view(torch.float64 if t.dtype == torch.complex128 else torch.float32)


@pytest.mark.parametrize("precision", BOTH)
@pytest.mark.parametrize("kind", ["separable", "rotor", "truncated"])
def test_noalloc_equals_plan_eval_two_calls(ctx, kind, precision):
    import torch
    if kind == "separable":
        big = scenes.airy_scene(64, npix=256, half_span_lamF=10.0)
        small = scenes.airy_scene(24, npix=96, npix_y=80)
    elif kind == "rotor":
        big = scenes.zernike_scene(7, n_across=40, npix=300, half_span=60e-6)
        small = scenes.zernike_scene(2404, n_across=24, npix=96, half_span=40e-6)
    else:
        big = scenes.truncated_airy_scene(40, npix=200, half_span_lamF=8.0)
        small = scenes.truncated_airy_scene(14, npix=90, npix_y=70, half_span_lamF=8.0)
    plans, refs, got = pair(ctx, big, small, precision)
    for sc, plan, r, g in zip((big, small), plans, refs, got):
        shape = plan.shape(precision)
        print(f"{kind} n={sc.n} px={sc.plane.nx}x{sc.plane.ny} precision={precision} shape={shape}", flush=True)
        assert torch.equal(bits(g), bits(r)), (kind, sc.n, precision)
    ref = oracle.eval_field(small)
    e = rel_l2(got[1].numpy(), ref)
    print(f"{kind} small vs oracle: {e:.2e}", flush=True)
    assert e <= TOL[precision]


@pytest.mark.parametrize("precision", BOTH)
def test_noalloc_lowers_an_automatic_segment_count_to_fit(ctx, precision):
    """The aberrated 1024 x 1024 workload: the rotor form's automatic 12
    segments would need 12 x 16 MiB of partials; the static 64 MiB buffer
    holds 4.  The allocation-free field equals gbd_plan_eval's at 4 segments
    bit for bit and the automatic one within the tolerance; a smaller input
    follows with its own automatic shape."""
    import torch
    big = scenes.config("zern128_1024")
    small = scenes.zernike_scene(2404, n_across=24, npix=96, half_span=40e-6)
    pb, ps = plan_of(ctx, big), plan_of(ctx, small)
    auto = pb.shape(precision)
    M = big.plane.nx * big.plane.ny
    assert auto["variant"] == 3 and auto["segments"] * M * 16 > LIMIT
    fit = dict(auto, segments=LIMIT // (M * 16))
    assert pb.shape(precision, opts=fit)["segments"] == fit["segments"]
    ref_auto = pb.eval(precision).cpu()
    ref_fit = pb.eval(precision, opts=fit).cpu()
    ref_small = ps.eval(precision).cpu()
    got = pb.eval_noalloc(precision)
    got_small = ps.eval_noalloc(precision)
    torch.cuda.synchronize()
    got, got_small = got.cpu(), got_small.cpu()
    assert torch.equal(bits(got), bits(ref_fit))
    assert torch.equal(bits(got_small), bits(ref_small))
    e = rel_l2(got.numpy(), ref_auto.numpy())
    print(f"zern128_1024 precision={precision}: {auto['segments']} -> {fit['segments']} segments, "
          f"vs automatic {e:.2e}", flush=True)
    assert e <= TOL[precision]


def test_noalloc_refuses_explicit_segments_beyond_the_buffer(ctx):
    """An explicit count whose partials exceed the static buffer is refused
    before any launch: the output keeps its contents."""
    import torch
    sc = scenes.config("zern128_1024")
    plan = plan_of(ctx, sc)
    out = torch.full((sc.plane.ny, sc.plane.nx), 3.0 + 1.0j, dtype=torch.complex64, device="cuda")
    with pytest.raises(gbd.GbdError) as e:
        plan.eval_noalloc(gbd.GBD_MIXED, out=out, opts=dict(segments=12))
    assert e.value.code == -7 and "static buffer" in str(e.value)
    torch.cuda.synchronize()
    assert bool((out == (3.0 + 1.0j)).all())
    # the count that fits is accepted and matches gbd_plan_eval
    o = dict(segments=4)
    ref = plan.eval(gbd.GBD_MIXED, opts=o)
    got = plan.eval_noalloc(gbd.GBD_MIXED, opts=o)
    torch.cuda.synchronize()
    assert torch.equal(bits(got.cpu()), bits(ref.cpu()))


def test_noalloc_empty_plan_clears_the_output(ctx):
    import torch
    sc = scenes.airy_scene(8, npix=5)
    empty = scenes.Scene(sc.lam, sc.l0, np.zeros((0, 2)), np.zeros((0, 2)), np.zeros(0) + 1e-3,
                         np.zeros((0, 2)), np.zeros(0), sc.abcd, sc.plane)
    plan = gbd.Plan(ctx, 16).setup(gbd.beamlets_from_scene(ctx, empty), gbd.plane_from_scene(ctx, empty))
    for prec, dt in ((gbd.GBD_MIXED, torch.complex64), (gbd.GBD_FP64, torch.complex128)):
        out = torch.full((5, 5), 2.0 - 1.0j, dtype=dt, device="cuda")
        plan.eval_noalloc(prec, out=out)
        torch.cuda.synchronize()
        assert not bool(out.abs().sum())


@pytest.mark.parametrize("precision,segments", [(gbd.GBD_MIXED, 20), (gbd.GBD_FP64, 10)])
def test_noalloc_refuses_explicit_segments_of_beamlets_in_rows(ctx, precision, segments):
    """Taken by rows no segment partials are written, but a count beyond the buffer stays refused, output untouched."""
    import torch
    sc = scenes.airy_scene(40, npix=700, npix_y=660, half_span_lamF=10.0)
    M = 700 * 660
    plan = plan_of(ctx, sc)
    most = LIMIT // (M * (8 if precision == gbd.GBD_MIXED else 16))
    assert segments > most
    out = torch.full((660, 700), 3.0 + 1.0j, dtype=plan.eval(precision).dtype, device="cuda")
    with pytest.raises(gbd.GbdError) as e:
        plan.eval_noalloc(precision, out=out, opts=dict(segments=segments))
    assert e.value.code == -7 and "static buffer" in str(e.value)
    torch.cuda.synchronize()
    assert bool((out == (3.0 + 1.0j)).all())
    got = plan.eval_noalloc(precision, opts=dict(segments=most - 1)).cpu()
    assert torch.equal(bits(got), bits(plan.eval(precision, opts=dict(segments=most - 1)).cpu()))
