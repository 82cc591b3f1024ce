"""Which kernel takes which call, by the kernels' names from the profiler: a
form that no longer ran would leave the accuracy tests passing on the form it
replaced.  Each case names the kernel that must have run; fields are held to
the FP64 oracle where another test does not do so at the same inputs."""
import re

import numpy as np
import pytest

import paper_2404_12454_amd as gbd
from paper_2404_12454_amd import scenes
from gbd_testutil import ensure_library

pytestmark = pytest.mark.gpu

F64, MIX = gbd.GBD_FP64, gbd.GBD_MIXED
ROTOR = r"eval_mixed_kernel<\d+, \d+, 2"  # form 2


@pytest.fixture(scope="module")
def ctx():
    ensure_library()
    return gbd.Context(0)


def kernels(call):
    """Names of the library's kernels that call() launches, template arguments and all."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    call()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    names = {e.name for e in p.events() if "gbd::" in e.name}
    if not names:
        pytest.skip("the profiler reports no kernels here")
    return {re.sub(r".*namespace\)::", "", n).split("(")[0] for n in names}


def permuted(sc):
    p = np.random.default_rng(1).permutation(sc.n)
    out = scenes.Scene(sc.lam, sc.l0, sc.r1[p], sc.th1[p], sc.w0[p], sc.amp[p], sc.path[p], sc.abcd, sc.plane)
    if sc.order is not None:
        out.order = sc.order[p]
    return out


def airy(nx=96, ny=66):
    return scenes.airy_scene(24, npix=nx, npix_y=ny, half_span_lamF=6.0)


def hermite(nx=96, ny=66):
    return scenes.hermite_scene(24, npix=nx, npix_y=ny, half_span_lamF=6.0)


def turned():
    sc = airy()
    sc.plane.xhint = np.array([0.0, 1.0, 0.0])  # a quarter turn: the rows lie along the detector's columns
    return sc


def weak(pitch, nx=200, ny=180, across=40):
    sc = scenes.zernike_scene(11, n_across=across, npix=nx, half_span=0.5 * nx * pitch)
    sc.plane.ny = ny
    return sc


def strong():
    sc = weak(0.1e-6)
    lens = np.eye(4)
    lens[2, 1] = lens[3, 0] = 5.0
    sc.abcd = np.ascontiguousarray((sc.abcd.reshape(-1, 4, 4) @ lens).reshape(-1, 16))
    return sc


def rim(across, nx, ny, span):
    return scenes.truncated_airy_scene(across, npix=nx, npix_y=ny, half_span_lamF=span)


ROUTES = [
    # rows: column blocks of one and two columns a lane, FP64 of one and eight
    (lambda: airy(64), MIX, None, "row_sum32_kernel<false, 1>"), (airy, MIX, None, "row_sum32_kernel<false, 2>"),
    (airy, F64, None, "row_sum64_kernel<false, 1>"), (lambda: airy(200), F64, None, "row_sum64_kernel<false, 8>"),
    (hermite, MIX, None, "row_sum32_kernel<true, 2>"), (hermite, F64, None, "row_sum64_kernel<true, 1>"),
    (lambda: hermite(200), F64, None, "row_sum64_kernel<true, 8>"), (airy, MIX, dict(segments=1, variant=4), "row_product_kernel"),
    # by beamlet: no order, a turned detector, the FP32 form
    (lambda: permuted(airy()), MIX, None, "eval_seph_kernel"), (turned, MIX, None, "eval_seph_kernel"),
    (lambda: permuted(airy()), F64, None, "eval_sep64_kernel"), (turned, F64, None, "eval_sep64_kernel"),
    (lambda: permuted(hermite()), MIX, None, "eval_seph_kernel"), (airy, MIX, dict(variant=5), "eval_sep_kernel"),
    # weak cross terms: both levels; the rotor form for one segment, another shape, long sums, strong terms, FP64
    (lambda: weak(0.05e-6), MIX, None, "eval_cross_kernel<1>"), (lambda: weak(0.15e-6), MIX, None, "eval_cross_kernel<2>"),
    (lambda: weak(0.1e-6, 127, 65), MIX, None, "eval_cross_kernel"), (lambda: weak(0.1e-6), MIX, dict(segments=2), "eval_cross_kernel"),
    (lambda: weak(0.1e-6), MIX, dict(segments=1), ROTOR), (lambda: weak(0.1e-6, across=64), MIX, dict(segments=2), ROTOR),
    (lambda: weak(0.1e-6), MIX, dict(rows_per_lane=16, waves=4), ROTOR), (strong, MIX, None, ROTOR),
    (lambda: weak(0.1e-6), F64, None, "eval_fp64_rotor_kernel"), (lambda: weak(0.1e-6, 64, 30), MIX, None, ROTOR),
    # truncated beamlets: every level of the columns, and pixel by pixel
    (lambda: rim(60, 66, 70, 0.8), MIX, None, "cut_column_mixed_kernel<32, 5, true>"),
    (lambda: rim(60, 66, 70, 1.2), MIX, None, "cut_column_mixed_kernel<16, 5, false>"),
    (lambda: rim(60, 65, 33, 1.0), MIX, None, "cut_column_mixed_kernel<16, 9, false>"),
    (lambda: rim(24, 63, 65, 4.0), MIX, None, "cut_column_mixed_kernel<8, 9, false>"),
    (lambda: rim(24, 100, 31, 4.0), MIX, None, "eval_cut_mixed_kernel"),
    (lambda: rim(60, 66, 70, 0.8), MIX, dict(variant=1), "eval_cut_mixed_kernel"),
    (lambda: rim(60, 66, 70, 0.8), F64, None, "cut_column_fp64_kernel<16, 9>"),
    (lambda: rim(60, 65, 33, 1.0), F64, None, "cut_column_fp64_kernel<16, 15>"),
    (lambda: rim(24, 63, 65, 4.0), F64, None, "cut_column_fp64_kernel<8, 15>"),
    (lambda: rim(24, 100, 31, 4.0), F64, None, "eval_cut_fp64_kernel"),
]


@pytest.mark.parametrize("make,precision,opts,kernel", ROUTES, ids=[f"{i}-{r[3].split('<')[0]}" for i, r in enumerate(ROUTES)])
def test_evaluations(ctx, make, precision, opts, kernel):
    import oracle
    from gbd_testutil import rel_l2
    sc = make()
    b, p = gbd.beamlets_from_scene(ctx, sc), gbd.plane_from_scene(ctx, sc)
    ran = kernels(lambda: gbd.gbd_eval(ctx, b, p, precision, opts=opts))
    assert sum(bool(re.match(kernel, k)) for k in ran) == 1, ran
    E = gbd.gbd_eval(ctx, b, p, precision, opts=opts).cpu().numpy()
    assert rel_l2(E, oracle.eval_field(sc)) <= (1e-12 if precision == F64 else 1e-6)


@pytest.mark.parametrize("count,make,kernel", [(1, airy, "batch_row_product_kernel"), (400, airy, "batch_row_product_wave_kernel<false>"),
                                               (2, lambda: permuted(airy()), "batch_sep_kernel"), (2, strong, r"batch_eval_kernel<\d+, \d+, 2>")])
def test_batches(ctx, count, make, kernel):
    sc = make()
    b, p = gbd.beamlets_from_scene(ctx, sc), gbd.plane_from_scene(ctx, sc)
    ran = kernels(lambda: gbd.gbd_eval_batch(ctx, [b] * count, [p] * count, fields=True))
    assert sum(bool(re.match(kernel, k)) for k in ran) == 1, ran


@pytest.mark.parametrize("mode,width,depth,kernel", [(gbd.GBD_MLP_BF16, 128, 3, "mlp_rows_kernel<3, 1, true>"),
                                                     (gbd.GBD_MLP_BF16, 256, 4, "mlp_rows_kernel<4, 2, true>"),
                                                     (gbd.GBD_MLP_BF16, 300, 2, "gemm"), (gbd.GBD_MLP_FP32, 128, 3, "gemm")])
def test_networks(ctx, mode, width, depth, kernel):
    import torch
    from paper_2404_12454_amd import surrogate
    net = gbd.Mlp(ctx, 5, width, depth, 32, mode)
    net.set_params(surrogate.init_params(width, depth, 5, seed=1))
    x, y = torch.randn(32, 5, device="cuda"), torch.randn(32, device="cuda")
    ran = kernels(lambda: net.backward(x, y))
    assert any(re.search(kernel, k) for k in ran), ran
