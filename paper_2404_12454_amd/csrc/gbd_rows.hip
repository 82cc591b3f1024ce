// Row-factored separable sum.
//
// A pupil grid is stored row by row, and through a system without cross
// terms the beamlets of a grid row land with one and the same y factor: same
// y of the base ray's hit point, same y slope, same y curvature.  Then
//   E(a, b) = sum_j U_j(a) V_j(b) = sum_c V_c(b) T_c(a),
//   T_c(a) = sum_{j in chunk c} U_j(a),
// every beamlet's x factor formed once per column (N nx phasors) and summed
// over its row, then a matrix product over the chunks.  The dense matrix
// form takes the product over all N beamlets.
//
// Row sums: a workgroup per (chunk, 64 C columns) whose 4 wavefronts take
//   every fourth beamlet each; a beamlet's record is uniform over the
//   wavefront (scalar loads, shared by C columns a lane), the factors are the
//   dense form's (FP64 phase, FP32 exp2/sin/cos) and are summed in FP32.  In
//   FP64 eight columns to a lane take two exponentials and then complex
//   multiplications, the factor's log being quadratic in x (row_sum64).
//   Bound by VALU issue.
//   The workgroups of a chunk also tabulate its y factors, once each.
// Products: 32 x 32 pixels per workgroup of 8 wavefronts that split the
//   chunks, MFMA with four real products (the sums are short, and Gauss's
//   three-product form would cost accuracy), the wavefronts' shares added in
//   FP64.
// Measured, a gbd_eval call of 51,468 beamlets on 512 x 512 pixels: mixed 310
// -> 45 us (row sums 25, product 10, setup 10) with an error against FP64 of
// 2e-7 instead of 9e-7, FP64 1,954 -> 73 us (50, 16, 10); the y factors formed
// by the product's tiles instead, nx / 32 times each: 46.5 and 79 us, of higher
// order 78 instead of 71.  441 instances of the parameter sweep 3.50 -> 1.27 ms
// (0.94 with the products by wavefronts and the host's share hidden).
#include "gbd_row_core.h"

namespace gbd {

namespace {

using namespace rows;

template <bool HG, int C>
__global__ void __launch_bounds__(64 * kRowSumWaves) row_sum32_kernel(RowGeom g, const int32_t *__restrict__ start,
                                                                      const Rec32 *__restrict__ rec,
                                                                      const RecHG32 *__restrict__ hg,
                                                                      const uint32_t *__restrict__ status,
                                                                      float2 *__restrict__ sums, StatusPost sp) {
    if (sp.post && blockIdx.x == 0 && threadIdx.x == 0) post_status(sp);
    row_sum_block32<HG, C>(g, blockIdx.x, start, rec, hg, status[1], sums);
}

template <bool HG, int C>
__global__ void __launch_bounds__(64 * kRowSumWaves) row_sum64_kernel(RowGeom g, const int32_t *__restrict__ start,
                                                                      const Rec64 *__restrict__ rec,
                                                                      const RecHG64 *__restrict__ hg,
                                                                      double2 *__restrict__ sums, StatusPost sp) {
    __shared__ double2 part[kRowSumWaves][64 * C];
    __shared__ double2 s2[kRowSumWaves][kRowLen / kRowSumWaves];
    if (sp.post && blockIdx.x == 0 && threadIdx.x == 0) post_status(sp);
    int c, x0;
    row_item<C>(blockIdx.x, g.nx, c, x0);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int j0 = start[c], j1 = start[c + 1];
    row_table<HG>(g, row_v64<HG>(rec[j0], HG ? hg + j0 : nullptr), c, x0, 64 * C, row_vtab(g, sums));
    int direct = 0;
    if constexpr (C > 1) {
        for (int i = threadIdx.x; i < j1 - j0; i += 64 * kRowSumWaves) {
            const Rec64 &r = rec[j0 + i];
            s2[i % kRowSumWaves][i / kRowSumWaves] = row_step64(r, g.dx);
            direct |= !(fabs(r.l[3]) * g.dx * g.dx <= kRowCurvature);
        }
        direct = __syncthreads_or(direct);
    }
    double2 t[C];
    row_sum64<HG, C>(rec, hg, j0 + w, j1, kRowSumWaves, g.a0 + (x0 + C * lane) * g.dx, g.dx, s2[w], direct != 0, t);
#pragma unroll
    for (int k = 0; k < C; k++) part[w][C * lane + k] = t[k];
    __syncthreads();
    for (int i = threadIdx.x; i < 64 * C && x0 + i < g.nx; i += 64 * kRowSumWaves) {
        double2 s = part[0][i];
#pragma unroll
        for (int k = 1; k < kRowSumWaves; k++) {
            s.x += part[k][i].x;
            s.y += part[k][i].y;
        }
        sums[(int64_t)c * g.nx + x0 + i] = s;
    }
}

// key: the FP32 sums' scale 2^-P, undone at the store (null in FP64)
template <typename R2>
__global__ void __launch_bounds__(64 * kRowWaves) row_product_kernel(RowGeom g, const R2 *__restrict__ sums,
                                                                     const uint32_t *__restrict__ status,
                                                                     R2 *__restrict__ out, EvalGuard gd) {
    __shared__ R2 part[kRowWaves][256 * kFoldBlocks<R2>];
    if (!guard_holds(gd)) return;
    const int tx = (g.nx + kRowTile - 1) / kRowTile, ty = (g.ny + kRowTile - 1) / kRowTile;
    const int w = work_item(blockIdx.x, gridDim.x);
    if (w >= tx * ty) return;
    // column strips, so that the workgroups of one XCD read few of the sums
    const int x0 = (w / ty) * kRowTile, y0 = (w % ty) * kRowTile;
    typename RowType<R2>::A4 re[2][2], im[2][2];
    row_product(sums, row_vtab(g, sums), g.chunks, g.nx, g.ny, x0, y0, re, im);
    const int P = status ? (int)row_exponent(status[1]) : 0;
    row_fold<R2>(re, im, part, [&](int p, int q, int i, double sr, double si) {
        const int ix = x0 + 16 * q + (i & 15), iy = y0 + 16 * p + (i >> 4);
        if (ix >= g.nx || iy >= g.ny) return;
        if constexpr (sizeof(R2) == sizeof(float2))
            out[(int64_t)iy * g.nx + ix] = row_value(sr, si, P);
        else
            out[(int64_t)iy * g.nx + ix] = make_double2(sr, si);
    });
}

dim3 row_sum_grid(const RowGeom &g, int c) { return dim3((unsigned)(g.chunks * ((g.nx + 64 * c - 1) / (64 * c)))); }
dim3 row_product_grid(const RowGeom &g) {
    const int64_t n = (int64_t)((g.nx + kRowTile - 1) / kRowTile) * ((g.ny + kRowTile - 1) / kRowTile);
    return dim3((unsigned)((n + 7) / 8 * 8));
}

}  // namespace

hipError_t launch_rows32(const RowGeom &g, const int32_t *start, const Rec32 *rec, const RecHG32 *hg,
                         const uint32_t *status, float2 *sums, float2 *out, const EvalGuard &guard,
                         hipStream_t s, hipEvent_t t0, hipEvent_t t1, const StatusPost &sp) {
    if (g.chunks < 1 || g.nx < 1 || g.ny < 1 || !status) return hipErrorInvalidValue;
    hipError_t e = g.nx > 64 ? launch_timed(hg ? row_sum32_kernel<true, 2> : row_sum32_kernel<false, 2>,
                                            row_sum_grid(g, 2), dim3(64 * kRowSumWaves), s, t0, nullptr, g, start, rec,
                                            hg, status, sums, sp)
                             : launch_timed(hg ? row_sum32_kernel<true, 1> : row_sum32_kernel<false, 1>,
                                            row_sum_grid(g, 1), dim3(64 * kRowSumWaves), s, t0, nullptr, g, start, rec,
                                            hg, status, sums, sp);
    if (e != hipSuccess) return e;
    return launch_timed(row_product_kernel<float2>, row_product_grid(g), dim3(64 * kRowWaves), s, nullptr, t1, g, sums,
                        status, out, guard);
}

hipError_t launch_rows64(const RowGeom &g, const int32_t *start, const Rec64 *rec, const RecHG64 *hg, double2 *sums,
                         double2 *out, const EvalGuard &guard, hipStream_t s, hipEvent_t t0, hipEvent_t t1,
                         const StatusPost &sp) {
    if (g.chunks < 1 || g.nx < 1 || g.ny < 1) return hipErrorInvalidValue;
    hipError_t e = g.nx > 192 ? launch_timed(hg ? row_sum64_kernel<true, 8> : row_sum64_kernel<false, 8>,
                                             row_sum_grid(g, 8), dim3(64 * kRowSumWaves), s, t0, nullptr, g, start,
                                             rec, hg, sums, sp)
                              : launch_timed(hg ? row_sum64_kernel<true, 1> : row_sum64_kernel<false, 1>,
                                             row_sum_grid(g, 1), dim3(64 * kRowSumWaves), s, t0, nullptr, g, start,
                                             rec, hg, sums, sp);
    if (e != hipSuccess) return e;
    return launch_timed(row_product_kernel<double2>, row_product_grid(g), dim3(64 * kRowWaves), s, nullptr, t1, g, sums,
                        (const uint32_t *)nullptr, out, guard);
}

}  // namespace gbd
