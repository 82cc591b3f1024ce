// Core of the row-factored separable sum, shared by the single evaluation
// and the batched sweep (see gbd_rows.hip for the method).
#pragma once

#include "gbd_sep_core.h"

namespace gbd {
namespace rows {

using namespace sep;

constexpr int kRowWaves = 8;      // wavefronts of a product workgroup, each a share of the chunks
constexpr int kRowTile = kRowTilePx;  // its pixel tile, 2 x 2 MFMA blocks
constexpr int kRowSumWaves = 4;   // wavefronts of a row-sum workgroup

__device__ inline float row_exponent(uint32_t key) { return key ? (float)((int)key - 2048) : 0.0f; }

// The words of a record that its x factor needs, uniform over the wavefront:
// two scalar loads (the unused words cost less than loads of their own).
typedef uint32_t u16w __attribute__((ext_vector_type(16), aligned(16)));
typedef uint32_t u8w __attribute__((ext_vector_type(8), aligned(16)));
struct RowWords {
    u16w a;
    u8w b;
    __device__ double f64(int k) const {
        const uint32_t lo = k < 16 ? a[k & 15] : b[k & 7], hi = k < 16 ? a[(k + 1) & 15] : b[(k + 1) & 7];
        return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
    }
    __device__ float f32(int k) const { return __builtin_bit_cast(float, (uint32_t)b[k & 7]); }
};
template <class Rec>
__device__ inline RowWords row_words(const Rec *__restrict__ r) {
    RowWords w;
    w.a = *reinterpret_cast<const u16w *>(r);
    w.b = *(reinterpret_cast<const u8w *>(r) + 2);
    return w;
}
static_assert(offsetof(Rec32, p) == 16 && offsetof(Rec32, m) == 64, "RowWords, Rec32");
static_assert(offsetof(Rec64, p) == 16 && offsetof(Rec64, l) == 64, "RowWords, Rec64");

// T(x) of one chunk at the lane's columns: the x factors of beamlets j0,
// j0 + step, ... < j1 summed in order in FP32 (a quarter of a chunk), every
// factor scaled by 2^ls.  C columns per lane share each record's loads.
template <bool HG, int C>
__device__ inline void row_sum32(const Rec32 *__restrict__ rec, const RecHG32 *__restrict__ hg, int j0, int j1,
                                 int step, const double (&ax)[C], float ls, float2 (&t)[C]) {
#pragma unroll
    for (int k = 0; k < C; k++) t[k] = make_float2(0.0f, 0.0f);
    if (j0 >= j1) return;
    RowWords w = row_words(rec + j0);
    for (int j = j0; j < j1; j += step) {
        const RowWords r = w;
        w = row_words(rec + min(j + step, j1 - 1));  // the next one's, in flight during this one's factors
        __builtin_amdgcn_sched_barrier(0);
        const double arho = r.f64(0), p0 = r.f64(4), p1 = r.f64(6), p3 = r.f64(10);
        const float m0 = r.f32(16) + ls, m1 = r.f32(17), m3 = r.f32(19);
#pragma unroll
        for (int k = 0; k < C; k++) {
            float ur, ui;
            const double d = ax[k] - arho;
            const float df = (float)d;  // rounded once: a pixel and a hit point each in FP32 would lose their difference
            factor(d, df, p0, p1, p3, m0, m1, m3, ur, ui);
            if constexpr (HG) {
                const RecHG32 *h = hg + j;
                hg_axis(df, h->g[0][0][0], h->g[0][0][1], h->cx0[0], h->cx0[1], h->cx1, h->cx2, ur, ui);
            }
            t[k].x += ur;
            t[k].y += ui;
        }
    }
}

// The same in FP64 over C consecutive columns a pitch dx apart.  With C > 1
// only the first column's factor and the ratio to the second are formed from
// exponentials; the factor's log is quadratic in x, so from there the factor
// is multiplied by the ratio and the ratio by the constant s2[i] of the
// wavefront's i-th beamlet (row_step64).  As in the FP64 rotor form this
// takes a well-sampled grid, |curvature| at most kRowCurvature per column^2,
// and caps the ln-amplitude slope at +-40 per column (a slope of 40 then puts
// the beamlet's peak over 280 columns away and the factor below e^-5000, zero
// either way); otherwise (direct) every column's factor is formed by itself.
template <bool HG, int C>
__device__ inline void row_sum64(const Rec64 *__restrict__ rec, const RecHG64 *__restrict__ hg, int j0, int j1,
                                 int step, double ax, double dx, const double2 *s2, bool direct, double2 (&t)[C]) {
#pragma unroll
    for (int k = 0; k < C; k++) t[k] = make_double2(0.0, 0.0);
    if (j0 >= j1) return;
    RowWords w = row_words(rec + j0);
    for (int j = j0, i = 0; j < j1; j += step, i++) {
        const RowWords r = w;
        w = row_words(rec + min(j + step, j1 - 1));
        __builtin_amdgcn_sched_barrier(0);
        const double d = ax - r.f64(0), p1 = r.f64(6), p3 = r.f64(10), l1 = r.f64(18), l3 = r.f64(22);
        double2 u = factor64(d, r.f64(4), p1, p3, r.f64(16), l1, l3);
        double2 q = make_double2(0.0, 0.0), s = q;
        if constexpr (C > 1) {
            double T = dx * (p1 + p3 * (2.0 * d + dx));
            T -= rint(T);
            q = cexp_turns64(fmin(fmax(dx * (l1 + l3 * (2.0 * d + dx)), -40.0), 40.0), T);
            s = s2[i];
        }
#pragma unroll
        for (int k = 0; k < C; k++) {
            double2 v = u;
            if constexpr (HG) {
                const RecHG64 *h = hg + j;
                v = hg_axis64(u, d + k * dx, h->g[0][0][0], h->g[0][0][1], h->cx0[0], h->cx0[1], h->cx1, h->cx2);
            }
            t[k].x += v.x;
            t[k].y += v.y;
            if (C > 1 && direct) {
                u = factor64(d + (k + 1) * dx, r.f64(4), p1, p3, r.f64(16), l1, l3);
            } else if (k + 1 < C) {
                u = make_double2(u.x * q.x - u.y * q.y, u.x * q.y + u.y * q.x);
                if (k + 2 < C) q = make_double2(q.x * s.x - q.y * s.y, q.x * s.y + q.y * s.x);
            }
        }
    }
}
constexpr double kRowCurvature = 0.07;  // ln amplitude per column^2
// e^(2 c dx^2), c the x factor's complex curvature: the ratio of successive
// ratios along a row
__device__ inline double2 row_step64(const Rec64 &r, double dx) {
    double T = 2.0 * r.p[3] * dx * dx;
    T -= rint(T);
    return cexp_turns64(2.0 * r.l[3] * dx * dx, T);
}

// A chunk's y factor (lv0: log2 of its scale, minus the bound of its modulus
// over the grid rows).
struct RowV32 {
    double brho, p2, p5;
    float m2, m5, lv0;
    float gyr, gyi, cy0r, cy0i, cy1, cy2;
};
struct RowV64 {
    double brho, p2, p5, l2, l5;
    double gyr, gyi, cy0r, cy0i, cy1, cy2;
};
// The chunk's y factor from its first beamlet's record.  lv0 = minus the
// bound of log2 |V| over the grid rows, so |V| 2^lv0 <= 1; the x factors
// take the rest of the common scale, 2^(-lv0 - P), 2^P the largest term over
// the grid: |U| 2^(-lv0 - P) <= 1 too, and a term lost to FP32's range lies
// 2^126 below the largest.
template <bool HG>
__device__ inline RowV32 row_v32(const Rec32 &r, const RecHG32 *h, double b0, double dy, int ny) {
    RowV32 v;
    v.brho = r.brho;
    v.p2 = r.p[2];
    v.p5 = r.p[5];
    v.m2 = r.m[2];
    v.m5 = r.m[5];
    double b;
    if constexpr (HG) {
        v.gyr = h->g[1][1][0];
        v.gyi = h->g[1][1][1];
        v.cy0r = h->cy0[0];
        v.cy0i = h->cy0[1];
        v.cy1 = h->cy1;
        v.cy2 = h->cy2;
        b = log2_hg_envelope_max(v.m2, v.m5, b0 - v.brho, dy, ny, hypotf(v.cy0r, v.cy0i), fabsf(v.cy1), fabsf(v.cy2),
                                 hypotf(v.gyr, v.gyi));
    } else {
        v.gyr = v.gyi = v.cy0r = v.cy0i = v.cy1 = v.cy2 = 0.0f;
        b = log2_envelope_max(v.m2, v.m5, b0 - v.brho, dy, ny);
    }
    v.lv0 = isfinite(b) ? -(float)b : 0.0f;
    return v;
}

template <bool HG>
__device__ inline RowV64 row_v64(const Rec64 &r, const RecHG64 *h) {
    RowV64 v = {};
    v.brho = r.brho;
    v.p2 = r.p[2];
    v.p5 = r.p[5];
    v.l2 = r.l[2];
    v.l5 = r.l[5];
    if constexpr (HG) {
        v.gyr = h->g[1][1][0];
        v.gyi = h->g[1][1][1];
        v.cy0r = h->cy0[0];
        v.cy0i = h->cy0[1];
        v.cy1 = h->cy1;
        v.cy2 = h->cy2;
    }
    return v;
}

template <bool HG>
__device__ inline float2 row_factor(const RowV32 &v, double by) {
    float vr, vi;
    const double d = by - v.brho;
    const float df = (float)d;
    factor(d, df, 0.0, v.p2, v.p5, v.lv0, v.m2, v.m5, vr, vi);
    if constexpr (HG) hg_axis(df, v.gyr, v.gyi, v.cy0r, v.cy0i, v.cy1, v.cy2, vr, vi);
    return make_float2(vr, vi);
}
template <bool HG>
__device__ inline double2 row_factor(const RowV64 &v, double by) {
    const double d = by - v.brho;
    double2 f = factor64(d, 0.0, v.p2, v.p5, 0.0, v.l2, v.l5);
    if constexpr (HG) f = hg_axis64(f, d, v.gyr, v.gyi, v.cy0r, v.cy0i, v.cy1, v.cy2);
    return f;
}

// A workgroup's (chunk, column block of 64 C) from its index
template <int C>
__device__ inline void row_item(int b, int nx, int &c, int &x0) {
    const int nb = (nx + 64 * C - 1) / (64 * C);
    c = b / nb;
    x0 = (b - c * nb) * 64 * C;
}

// The y factors [chunks][ny] lie behind the row sums [chunks][nx].
template <typename R2>
__host__ __device__ inline R2 *row_vtab(const RowGeom &g, R2 *sums) { return sums + (int64_t)g.chunks * g.nx; }

// The chunk's y factors over the grid rows, shared out over the workgroups of
// its column blocks (`cols` columns each): once each, where the tiles of the
// product would form them nx / 32 times.
template <bool HG, typename V, typename R2>
__device__ inline void row_table(const RowGeom &g, const V &v, int c, int x0, int cols, R2 *__restrict__ vtab) {
    const int nb = (g.nx + cols - 1) / cols, per = (g.ny + nb - 1) / nb, k = x0 / cols;
    for (int y = k * per + threadIdx.x; y < min(g.ny, (k + 1) * per); y += 64 * kRowSumWaves)
        vtab[(int64_t)c * g.ny + y] = row_factor<HG>(v, g.b0 + y * g.dy);
}

// Workgroup b of the FP32 row sums: its wavefronts take every fourth beamlet
// of the chunk each, and their sums are added in order.  key: the setup's
// (largest term).
template <bool HG, int C>
__device__ inline void row_sum_block32(const RowGeom &g, int b, const int32_t *__restrict__ start,
                                       const Rec32 *__restrict__ rec, const RecHG32 *__restrict__ hg, uint32_t key,
                                       float2 *__restrict__ sums) {
    __shared__ float2 part[kRowSumWaves][64 * C];
    int c, x0;
    row_item<C>(b, g.nx, c, x0);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int j0 = start[c], j1 = start[c + 1];
    const RowV32 rv = row_v32<HG>(rec[j0], HG ? hg + j0 : nullptr, g.b0, g.dy, g.ny);
    row_table<HG>(g, rv, c, x0, 64 * C, row_vtab(g, sums));
    double ax[C];
    float2 t[C];
#pragma unroll
    for (int k = 0; k < C; k++) ax[k] = g.a0 + (x0 + 64 * k + lane) * g.dx;
    row_sum32<HG, C>(rec, hg, j0 + w, j1, kRowSumWaves, ax, -rv.lv0 - row_exponent(key), t);
#pragma unroll
    for (int k = 0; k < C; k++) part[w][64 * k + lane] = t[k];
    __syncthreads();
    for (int i = threadIdx.x; i < 64 * C && x0 + i < g.nx; i += 64 * kRowSumWaves) {
        float2 s = part[0][i];
#pragma unroll
        for (int k = 1; k < kRowSumWaves; k++) {
            s.x += part[k][i].x;
            s.y += part[k][i].y;
        }
        sums[(int64_t)c * g.nx + x0 + i] = s;
    }
}

__device__ inline f4 row_mfma(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ inline d4 row_mfma(double a, double b, d4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

template <typename R2>
struct RowType;
template <>
struct RowType<float2> {
    using R = float;
    using A4 = f4;
    // row of element e of a result block
    __device__ static int row(int lk, int e) { return 4 * lk + e; }
};
template <>
struct RowType<double2> {
    using R = double;
    using A4 = d4;
    __device__ static int row(int lk, int e) { return lk + 4 * e; }
};

// One wavefront's share of the product for the 32 x 32 tile at (x0, y0):
// steps of four chunks (the MFMA's K) w, w + kRowWaves, ... of the
// workgroup's wavefront w.  Lane l holds chunk 4 step + l / 16: its y factor
// at rows 16 p + l % 16 as the A operand, its row sum at columns
// 16 q + l % 16 as the B operand.  Four real products per complex one.
// Chunks past the end and pixels past the grid read a clamped element and
// count as zero / are not stored.
template <typename R2>
__device__ inline void row_product(const R2 *__restrict__ sums, const R2 *__restrict__ vtab, int chunks, int nx, int ny,
                                   int x0, int y0, typename RowType<R2>::A4 (&re)[2][2],
                                   typename RowType<R2>::A4 (&im)[2][2]) {
    using R = typename RowType<R2>::R;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
    int xc[2], yc[2];
#pragma unroll
    for (int p = 0; p < 2; p++) {
        yc[p] = min(y0 + 16 * p + li, ny - 1);
        xc[p] = min(x0 + 16 * p + li, nx - 1);
    }
#pragma unroll
    for (int p = 0; p < 2; p++)
#pragma unroll
        for (int q = 0; q < 2; q++) re[p][q] = im[p][q] = typename RowType<R2>::A4{0, 0, 0, 0};
    const int steps = (chunks + 3) >> 2;
    auto load = [&](int s, R2 (&f)[2], R2 (&t)[2]) {
        const int c = 4 * s + lk, cc = min(c, chunks - 1);
#pragma unroll
        for (int q = 0; q < 2; q++) {
            f[q] = vtab[(int64_t)cc * ny + yc[q]];
            t[q] = sums[(int64_t)cc * nx + xc[q]];
            if (c >= chunks) t[q].x = t[q].y = R(0);
        }
    };
    if (w >= steps) return;
    R2 fn[2], tn[2];
    load(w, fn, tn);
    for (int s = w; s < steps; s += kRowWaves) {
        const R2 f[2] = {fn[0], fn[1]}, t[2] = {tn[0], tn[1]};
        load(min(s + kRowWaves, steps - 1), fn, tn);  // the next step's, used after this one's products
#pragma unroll
        for (int p = 0; p < 2; p++)
#pragma unroll
            for (int q = 0; q < 2; q++) {
                re[p][q] = row_mfma(f[p].x, t[q].x, re[p][q]);
                im[p][q] = row_mfma(f[p].x, t[q].y, im[p][q]);
                re[p][q] = row_mfma(-f[p].y, t[q].y, re[p][q]);
                im[p][q] = row_mfma(f[p].y, t[q].x, im[p][q]);
            }
    }
}

// The workgroup's shares added in wavefront order in FP64, a row of two
// 16 x 16 blocks at a time through LDS in FP32 (FP64: one block, for 32 KiB of
// LDS either way); pixel(p, q, i, value) gets element i (row i / 16, column
// i % 16) of block (p, q) from one thread.
template <typename R2>
constexpr int kFoldBlocks = sizeof(R2) == sizeof(float2) ? 2 : 1;
template <typename R2, typename F>
__device__ inline void row_fold(typename RowType<R2>::A4 (&re)[2][2], typename RowType<R2>::A4 (&im)[2][2],
                                R2 (*part)[256 * kFoldBlocks<R2>], F pixel) {
    constexpr int N = kFoldBlocks<R2>;
    static_assert(256 * N <= 64 * kRowWaves, "a thread per pixel");
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
#pragma unroll
    for (int p = 0; p < 2; p++)
#pragma unroll
        for (int q0 = 0; q0 < 2; q0 += N) {
            __syncthreads();
#pragma unroll
            for (int q = 0; q < N; q++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    R2 x;
                    x.x = re[p][q0 + q][e];
                    x.y = im[p][q0 + q][e];
                    part[w][256 * q + 16 * RowType<R2>::row(lk, e) + li] = x;
                }
            __syncthreads();
            if (threadIdx.x < 256 * N) {
                double sr = 0.0, si = 0.0;
#pragma unroll
                for (int k = 0; k < kRowWaves; k++) {
                    const R2 x = part[k][threadIdx.x];
                    sr += (double)x.x;
                    si += (double)x.y;
                }
                pixel(p, q0 + (int)(threadIdx.x >> 8), (int)threadIdx.x & 255, sr, si);
            }
        }
}

// The whole product of a 32 x 32 tile by one wavefront, bit for bit the
// workgroup's: each of its kRowWaves shares in FP32, in the same step order,
// then added in FP64 in the shares' order.  Element e of block (p, q) is row
// 4 (lane / 16) + e, column lane % 16.
__device__ inline void row_product_wave(const float2 *__restrict__ sums, const float2 *__restrict__ vtab, int chunks,
                                        int nx, int ny, int x0, int y0, double (&sr)[2][2][4],
                                        double (&si)[2][2][4]) {
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int xc[2] = {min(x0 + li, nx - 1), min(x0 + 16 + li, nx - 1)};
    const int yc[2] = {min(y0 + li, ny - 1), min(y0 + 16 + li, ny - 1)};
    const int steps = (chunks + 3) >> 2;
    auto load = [&](int s, float2 (&f)[2], float2 (&t)[2]) {
        const int c = 4 * s + lk, cc = min(c, chunks - 1);
#pragma unroll
        for (int q = 0; q < 2; q++) {
            f[q] = vtab[(int64_t)cc * ny + yc[q]];
            t[q] = sums[(int64_t)cc * nx + xc[q]];
            if (c >= chunks) t[q].x = t[q].y = 0.0f;
        }
    };
#pragma unroll
    for (int p = 0; p < 2; p++)
#pragma unroll
        for (int q = 0; q < 2; q++)
#pragma unroll
            for (int e = 0; e < 4; e++) sr[p][q][e] = si[p][q][e] = 0.0;
    float2 fn[2], tn[2];
    if (steps > 0) load(0, fn, tn);
    for (int w = 0; w < min(kRowWaves, steps); w++) {  // a share without steps adds zero
        f4 re[2][2], im[2][2];
#pragma unroll
        for (int p = 0; p < 2; p++)
#pragma unroll
            for (int q = 0; q < 2; q++) re[p][q] = im[p][q] = f4{0, 0, 0, 0};
        for (int s = w; s < steps; s += kRowWaves) {
            const float2 f[2] = {fn[0], fn[1]}, t[2] = {tn[0], tn[1]};
            load(min(s + kRowWaves < steps ? s + kRowWaves : w + 1, steps - 1), fn, tn);
#pragma unroll
            for (int p = 0; p < 2; p++)
#pragma unroll
                for (int q = 0; q < 2; q++) {
                    re[p][q] = row_mfma(f[p].x, t[q].x, re[p][q]);
                    im[p][q] = row_mfma(f[p].x, t[q].y, im[p][q]);
                    re[p][q] = row_mfma(-f[p].y, t[q].y, re[p][q]);
                    im[p][q] = row_mfma(f[p].y, t[q].x, im[p][q]);
                }
        }
#pragma unroll
        for (int p = 0; p < 2; p++)
#pragma unroll
            for (int q = 0; q < 2; q++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    sr[p][q][e] += (double)re[p][q][e];
                    si[p][q][e] += (double)im[p][q][e];
                }
    }
}

// The FP32 sums' scale 2^-P undone
__device__ inline float2 row_value(double sr, double si, int P) {
    return make_float2((float)ldexp(sr, P), (float)ldexp(si, P));
}

}  // namespace rows
}  // namespace gbd
