// Matrix form for beamlets with weak cross terms, mixed precision.
//
// On a tilted detector or behind an aberrated system a beamlet's phasor has
// a cross term x da db (x complex), so the sum over the beamlets does not
// separate by the plane's axes.  Within one 128 x 128 pixel tile it nearly
// does: about the tile's centre (a_c, b_c), a = a_c + u, b = b_c + v,
//   x da db = x da db_c + x da_c v + x u v,
// whose first two terms belong to one axis each and go into the factors U
// and V, and the rest is small (a spot is many tiles wide: |x u v| is 1e-3
// in the corner of a tile on the f/4 aberrated 1024 x 1024 workload), so
// e^(x u v) is its series, each term again a product of one factor per axis:
//   sum_j U_j V_j (1 + (x_j u) v + (x_j u)^2/2 v^2 + ...)
// on FP16 MFMA in hi/lo halves, as the separable form.  The setup bounds |x|
// at the corner over all beamlets (FLAG_CROSS1, FLAG_CROSS2): up to 2^-10
// one further product of the leading halves does (8 MFMAs per 16 beamlets
// and 16 x 16 block, 6 without cross terms), up to 2^-6 fourteen, beyond the
// rotor form is kept.  Truncation and rounding of the small products are
// below 1e-7 of a term (root mean square over a tile) at those limits.
//
// 12,892 beamlets on 1024 x 1024 pixels: a gbd_eval call 2,678 us (rotor) ->
// 487 us, error against FP64 5.0e-7 -> 4.6e-7; 12,720 traced ones on 512 x
// 512: the kernel 775 -> 127 us.  (Records read from LDS by every lane: 535
// and 146 us; with the factors ahead of the products as the scheduler chose
// besides: 570 and 160.)
// Bound by MFMA and the factors' VALU, which overlap little at two
// wavefronts per SIMD; a 128 x 128 tile (2 x 4 wavefronts of 64 x 32) keeps
// the series short and the operands within LDS.
#include "gbd_cross_core.h"

namespace gbd {

namespace {

using namespace cross;

template <int LEVEL>
__global__ void __launch_bounds__(kThreads) eval_cross_kernel(EvalGeom g, const Rec32 *__restrict__ rec,
                                                              const uint32_t *__restrict__ status,
                                                              float2 *__restrict__ partial, StatusPost sp) {
    __shared__ CrossLds<LEVEL> L;
    if (sp.post && blockIdx.x == 0 && threadIdx.x == 0) post_status(sp);
    const int w = work_item(blockIdx.x, gridDim.x);
    if (w >= g.work) return;
    const int tiles = g.tiles_x * g.tiles_y;
    const int seg = w / tiles, t = w - seg * tiles;
    const int ty = t / g.tiles_x, tx = t - ty * g.tiles_x;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    const SepGeom sg{g.nx, g.ny, g.a0, g.b0, g.dx, g.dy};
    const int64_t jb = (int64_t)seg * g.seg_len, je = min(g.n, jb + g.seg_len);
    const uint32_t key = status[1];
    const int P = key ? (int)key - 2048 : 0;
    f4 accR[kBY][kBX], accI[kBY][kBX];
    cross_accumulate<LEVEL>(sg, rec, jb, je, tx, ty, (float)P, L, accR, accI);
    const int64_t M = (int64_t)g.nx * g.ny;
    const int x0 = tx * kCrossTile + 16 * kBX * (wv % kWX), y0 = ty * kCrossTile + 16 * kBY * (wv / kWX);
    const int down = P - kUExp - kVExp;
#pragma unroll
    for (int p = 0; p < kBY; p++)
#pragma unroll
        for (int q = 0; q < kBX; q++) {
            const int ix = x0 + 16 * q + li;
            if (ix >= g.nx) continue;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int iy = y0 + 16 * p + 4 * lk + e;
                if (iy >= g.ny) continue;
                partial[(int64_t)seg * M + (int64_t)iy * g.nx + ix] =
                    make_float2(ldexpf(accR[p][q][e], down), ldexpf(accI[p][q][e], down));
            }
        }
}

}  // namespace

hipError_t launch_eval_cross(int level, const EvalGeom &g, const Rec32 *rec, const uint32_t *status, float2 *partial,
                             hipStream_t s, hipEvent_t t0, hipEvent_t t1, const StatusPost &sp) {
    if (!status || level < 1 || level > 2) return hipErrorInvalidValue;
    const dim3 grid((g.work + 7) / 8 * 8), block(kThreads);
    return launch_timed(level == 1 ? eval_cross_kernel<1> : eval_cross_kernel<2>, grid, block, s, t0, t1, g, rec, status,
                        partial, sp);
}

}  // namespace gbd
