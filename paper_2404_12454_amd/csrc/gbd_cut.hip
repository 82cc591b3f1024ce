// Truncated beamlets: a Gaussian beamlet whose input envelope is cut by a
// straight edge (kept where e . r <= t) arrives on a plane normal to the axis
// as its Gaussian field times erfc(zeta) / 2, zeta = z0 + za da + zb db (the
// setup kernel's RecCut record).  Direct form: every pixel of every cut
// beamlet forms the Gaussian phasor as the direct mixed (or FP64) form does
// and the complementary error function through the Faddeeva function
// w(u) = e^(-u^2) erfc(-i u):
//   Re zeta >= 0:  E erfc(zeta) / 2 = e^(log E - zeta^2) w(i zeta) / 2,
//   Re zeta <  0:  E erfc(zeta) / 2 = E - e^(log E - zeta^2) w(-i zeta) / 2,
// so the exponent log E - zeta^2 is formed before any exponential (each of
// e^(log E) and erfc(zeta) alone can under- or overflow where their product
// is finite) and w is only taken in the upper half plane, where |w| <= 1.  w
// by Weideman's rational approximation (FaddeevaCoef).  The cut beamlets are
// few (those near an aperture edge), so the others keep the fast forms and
// this kernel adds its segments to the same partial sums.
#include "gbd_device.h"

namespace gbd {

namespace {

using namespace dev;

// w(u) for Im u >= 0, FP32 (u = (ur, ui))
__device__ inline float2 faddeeva32(const FaddeevaCoef &fc, float ur, float ui) {
    const float L = fc.L32;
    // 1 / (L - i u) = 1 / ((L + ui) - i ur)
    const float dr = L + ui, di = -ur;
    const float inv = __builtin_amdgcn_rcpf(fmaf(dr, dr, di * di));
    const float vr = dr * inv, vi = -di * inv;
    // Z = (L + i u) / (L - i u) = ((L - ui) + i ur) v
    const float nr = L - ui, ni = ur;
    const float Zr = nr * vr - ni * vi, Zi = nr * vi + ni * vr;
    float pr = fc.a32[kFaddeevaN32 - 1], pi = 0.0f;
#pragma unroll
    for (int n = kFaddeevaN32 - 2; n >= 0; n--) {
        const float tr = fmaf(pr, Zr, fmaf(-pi, Zi, fc.a32[n]));
        pi = fmaf(pr, Zi, pi * Zr);
        pr = tr;
    }
    // w = v (2 p v + 1 / sqrt(pi))
    const float sr = fmaf(2.0f * pr, vr, fmaf(-2.0f * pi, vi, 0.56418958354775628f));
    const float si = 2.0f * (pr * vi + pi * vr);
    return make_float2(vr * sr - vi * si, vr * si + vi * sr);
}

__device__ inline cd faddeeva64(const FaddeevaCoef &fc, double ur, double ui) {
    const double L = fc.L64;
    const cd v = cdiv(mk(1.0, 0.0), mk(L + ui, -ur));
    const cd Z = mul(mk(L - ui, ur), v);
    cd p = mk(fc.a64[kFaddeevaN64 - 1], 0.0);
#pragma unroll
    for (int n = kFaddeevaN64 - 2; n >= 0; n--) p = add(mul(p, Z), mk(fc.a64[n], 0.0));
    return mul(v, add(scl(mul(p, v), 2.0), mk(0.56418958354775628695, 0.0)));
}

template <int ROWS, int WAVES>
__global__ void __launch_bounds__(64 * WAVES) eval_cut_mixed_kernel(EvalGeom g, const Rec32 *__restrict__ rec,
                                                                    const RecCut32 *__restrict__ cut,
                                                                    FaddeevaCoef fc, int32_t seg_base,
                                                                    float4 *__restrict__ partial) {
    __shared__ Rec32 tile[kMixedTile];
    __shared__ RecCut32 ctile[kMixedTile];
    const int w = work_item(blockIdx.x, gridDim.x);
    if (w >= g.work) return;
    const int tiles = g.tiles_x * g.tiles_y;
    const int seg = w / tiles;
    const int t = w - seg * tiles;
    const int ty = t / g.tiles_x, tx = t - ty * g.tiles_x;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int ix = tx * 64 + lane;
    const int iy0 = (ty * WAVES + wv) * ROWS;
    const double a = g.a0 + ix * g.dx;
    const double b0 = g.b0 + iy0 * g.dy;
    const double dy = g.dy, dy2 = g.dy * g.dy;
    const float af = (float)a, b0f = (float)b0, dyf = (float)dy;
    constexpr float kLog2e = 1.4426950408889634f, kInv2Pi = 0.15915494309189535f;

    float s_re[ROWS], s_im[ROWS], c_re[ROWS], c_im[ROWS], acc_re[ROWS], acc_im[ROWS];
#pragma unroll
    for (int k = 0; k < ROWS; k++) s_re[k] = s_im[k] = c_re[k] = c_im[k] = acc_re[k] = acc_im[k] = 0.0f;
    const int64_t jb = (int64_t)seg * g.seg_len;
    const int64_t je = min(g.n, jb + g.seg_len);
    for (int64_t j0 = jb; j0 < je; j0 += kMixedTile) {
        const int cnt = (int)min((int64_t)kMixedTile, je - j0);
        __syncthreads();
        {
            const float4 *src = reinterpret_cast<const float4 *>(rec + j0);
            float4 *dst = reinterpret_cast<float4 *>(tile);
            for (int i = threadIdx.x; i < cnt * kRec32Vec4; i += 64 * WAVES) dst[i] = src[i];
            const float4 *cs = reinterpret_cast<const float4 *>(cut + j0);
            float4 *cd4 = reinterpret_cast<float4 *>(ctile);
            for (int i = threadIdx.x; i < cnt * 2; i += 64 * WAVES) cd4[i] = cs[i];
        }
        __syncthreads();
        for (int jj = 0; jj < cnt; jj++) {
            const Rec32 &r = tile[jj];
            const RecCut32 &c = ctile[jj];
            const double da = a - r.arho, db = b0 - r.brho;
            const double q = r.p[2] + r.p[4] * da;
            const double T0 = r.p[0] + da * (r.p[1] + r.p[3] * da) + db * (q + r.p[5] * db);
            const double T1 = dy * (q + 2.0 * r.p[5] * db);
            const double T2 = r.p[5] * dy2;
            const float daf = af - r.arho_f, dbf0 = b0f - r.brho_f;
            const float qf = r.m[2] + r.m[4] * daf;
            const float Uc = r.m[0] + daf * (r.m[1] + r.m[3] * daf);
            const float zr0 = fmaf(c.za[0], daf, c.z0[0]), zi0 = fmaf(c.za[1], daf, c.z0[1]);
#pragma unroll
            for (int k = 0; k < ROWS; k++) {
                const double th = T0 + (double)k * (T1 + (double)k * T2);
                const float ph = (float)__builtin_amdgcn_fract(th);
                const float dbf = fmaf((float)k, dyf, dbf0);
                const float L = Uc + dbf * (qf + r.m[5] * dbf);
                // zeta, folded into the right half plane
                float zr = fmaf(c.zb[0], dbf, zr0), zi = fmaf(c.zb[1], dbf, zi0);
                const bool neg = zr < 0.0f;
                zr = neg ? -zr : zr;
                zi = neg ? -zi : zi;
                // e^(log E - zeta^2) / 2: log2-amplitude and phase in turns
                const float L2 = L - 1.0f - (zr * zr - zi * zi) * kLog2e;
                const float ph2 = __builtin_amdgcn_fractf(ph - 2.0f * zr * zi * kInv2Pi);
                const float m2 = __builtin_amdgcn_exp2f(L2);
                const float er = m2 * __builtin_amdgcn_cosf(ph2), ei = m2 * __builtin_amdgcn_sinf(ph2);
                const float2 W = faddeeva32(fc, -zi, zr);  // w(i zeta)
                float tr = er * W.x - ei * W.y, ti = er * W.y + ei * W.x;
                if (neg) {
                    const float m = __builtin_amdgcn_exp2f(L);
                    tr = m * __builtin_amdgcn_cosf(ph) - tr;
                    ti = m * __builtin_amdgcn_sinf(ph) - ti;
                }
                acc_re[k] += tr;
                acc_im[k] += ti;
            }
        }
#pragma unroll
        for (int k = 0; k < ROWS; k++) {
            kahan(s_re[k], c_re[k], acc_re[k]);
            kahan(s_im[k], c_im[k], acc_im[k]);
            acc_re[k] = acc_im[k] = 0.0f;
        }
    }
    if (ix >= g.nx) return;
    const int64_t M = (int64_t)g.nx * g.ny;
#pragma unroll
    for (int k = 0; k < ROWS; k++) {
        const int iy = iy0 + k;
        if (iy < g.ny)
            partial[(int64_t)(seg_base + seg) * M + (int64_t)iy * g.nx + ix] =
                make_float4(s_re[k], s_im[k], c_re[k], c_im[k]);
    }
}

template <int ROWS, int WAVES>
__global__ void __launch_bounds__(64 * WAVES) eval_cut_fp64_kernel(EvalGeom g, const Rec64 *__restrict__ rec,
                                                                   const RecCut64 *__restrict__ cut,
                                                                   FaddeevaCoef fc, int32_t seg_base,
                                                                   double2 *__restrict__ partial) {
    constexpr int CH = 64;
    __shared__ Rec64 tile[CH];
    __shared__ RecCut64 ctile[CH];
    const int w = work_item(blockIdx.x, gridDim.x);
    if (w >= g.work) return;
    const int tiles = g.tiles_x * g.tiles_y;
    const int seg = w / tiles;
    const int t = w - seg * tiles;
    const int ty = t / g.tiles_x, tx = t - ty * g.tiles_x;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int ix = tx * 64 + lane;
    const int iy0 = (ty * WAVES + wv) * ROWS;
    const double a = g.a0 + ix * g.dx;
    const double b0 = g.b0 + iy0 * g.dy;
    const double dy = g.dy, dy2 = g.dy * g.dy;

    double acc_re[ROWS], acc_im[ROWS];
#pragma unroll
    for (int k = 0; k < ROWS; k++) acc_re[k] = acc_im[k] = 0.0;
    const int64_t jb = (int64_t)seg * g.seg_len;
    const int64_t je = min(g.n, jb + g.seg_len);
    for (int64_t j0 = jb; j0 < je; j0 += CH) {
        const int cnt = (int)min((int64_t)CH, je - j0);
        __syncthreads();
        {
            const double2 *src = reinterpret_cast<const double2 *>(rec + j0);
            double2 *dst = reinterpret_cast<double2 *>(tile);
            for (int i = threadIdx.x; i < cnt * 8; i += 64 * WAVES) dst[i] = src[i];
            const double2 *cs = reinterpret_cast<const double2 *>(cut + j0);
            double2 *cd2 = reinterpret_cast<double2 *>(ctile);
            for (int i = threadIdx.x; i < cnt * 4; i += 64 * WAVES) cd2[i] = cs[i];
        }
        __syncthreads();
        for (int jj = 0; jj < cnt; jj++) {
            const Rec64 &r = tile[jj];
            const RecCut64 &c = ctile[jj];
            const double da = a - r.arho, db = b0 - r.brho;
            const double q = r.p[2] + r.p[4] * da;
            const double T0 = r.p[0] + da * (r.p[1] + r.p[3] * da) + db * (q + r.p[5] * db);
            const double T1 = dy * (q + 2.0 * r.p[5] * db);
            const double T2 = r.p[5] * dy2;
            const double ql = r.l[2] + r.l[4] * da;
            const double Vc = r.l[0] + da * (r.l[1] + r.l[3] * da);
#pragma unroll
            for (int k = 0; k < ROWS; k++) {
                const double th = T0 + (double)k * (T1 + (double)k * T2);
                const double rr = th - rint(th);
                const double dbk = fma((double)k, dy, db);
                const double lnm = Vc + dbk * (ql + r.l[5] * dbk);
                double zr = c.z0[0] + c.za[0] * da + c.zb[0] * dbk;
                double zi = c.z0[1] + c.za[1] * da + c.zb[1] * dbk;
                const bool neg = zr < 0.0;
                zr = neg ? -zr : zr;
                zi = neg ? -zi : zi;
                // e^(log E - zeta^2) / 2 (phase in turns)
                double ph2 = rr - zr * zi / kPi;
                ph2 -= rint(ph2);
                double s2, c2;
                sincospi(2.0 * ph2, &s2, &c2);
                const double m2 = 0.5 * exp(lnm - (zr * zr - zi * zi));
                const cd W = faddeeva64(fc, -zi, zr);
                double tr = m2 * (c2 * W.re - s2 * W.im), ti = m2 * (c2 * W.im + s2 * W.re);
                if (neg) {
                    double s, cc;
                    sincospi(2.0 * rr, &s, &cc);
                    const double m = exp(lnm);
                    tr = m * cc - tr;
                    ti = m * s - ti;
                }
                acc_re[k] += tr;
                acc_im[k] += ti;
            }
        }
    }
    if (ix >= g.nx) return;
    const int64_t M = (int64_t)g.nx * g.ny;
#pragma unroll
    for (int k = 0; k < ROWS; k++) {
        const int iy = iy0 + k;
        if (iy < g.ny)
            partial[(int64_t)(seg_base + seg) * M + (int64_t)iy * g.nx + ix] = make_double2(acc_re[k], acc_im[k]);
    }
}

// ---------------------------------------------------------------------------
// Column form.  Over the few rows of a lane's column erfc(zeta) hardly varies:
// with delta = zb dy the change of zeta per row, zeta_k = zeta_0 + k delta,
// the term is the rotor form's phasor times a short Taylor polynomial in k
// about the column's anchor row,
//   E_k erfc(zeta_k) / 2 = A rho^k sigma^(k^2) sum_p m_p k^p,
// so the complex error function, the phasor's transcendentals and the
// derivatives f' = -e^(-zeta^2) / sqrt(pi), f^(p+1) = -2 zeta f^(p) -
// 2 (p - 1) f^(p-1) are formed once per column.  The anchor A takes
// e^(-zeta_0^2) into its exponent where that keeps both factors bounded
// (Re zeta_0 >= 0, or Re zeta_0^2 < 0), else the polynomial does.
// For all pixels |m_p k^p| falls at least as (e t / p)^p with
// t = |k delta| (2 |zeta| + sqrt(2 p)); the setup bounds t over the cut
// beamlets and the grid (kCutReachLow, kCutReachHigh), where degrees 5 and 9
// leave 2^-25 of a term in FP32, 9 and 15 2^-50 in FP64: 16 rows (mixed 32
// where that reaches) at the low degree, else at the high one, else 8 rows;
// beyond that the direct form.
// Bound by VALU issue: at the low degree 510 instructions a column of 16
// pixels (32 a pixel) or 820 of 32 (26), the direct form about 130 a pixel.
// 2,028 cut beamlets on 512 x 512 pixels, mixed: the kernel 1,450 -> 430 us by
// 16 rows, 300 by 32 (the evaluation 1,762 -> 437, 325 us, error against FP64
// 7.7e-7 -> 1.8e-7, 1.4e-7); 512 on 256 x 256, FP64: 639 -> 142 us.
// 512 on 400 x 400, which needs the high degree: 16 rows 155 us, 8 rows 197.
// ---------------------------------------------------------------------------

// m_p, p = 0 ... DEG.  z: zeta_0 folded into the right half plane (neg: it
// was negated), w = w(i z), c = e^(zeta_0^2) if big else e^(-zeta_0^2) (used
// where neg), big: the anchor holds e^(-zeta_0^2); d = delta.
template <int DEG, typename R>
__device__ inline void edge_poly(R zr, R zi, bool neg, bool big, R wr, R wi, R cr, R ci, R dr, R di,
                                 R (&m)[DEG + 1][2]) {
    const R half = (R)0.5, n1 = (R)-0.56418958354775628695;  // -1 / sqrt(pi)
    const bool low = neg && !big;
    // neg: (big ? c : 1) - (big ? w : c w) / 2, else w / 2
    const R xr = low ? cr * wr - ci * wi : wr, xi = low ? cr * wi + ci * wr : wi;
    m[0][0] = neg ? (big ? cr : (R)1) - half * xr : half * xr;
    m[0][1] = neg ? (big ? ci : (R)0) - half * xi : half * xi;
    const R qr = low ? n1 * cr : n1, qi = low ? n1 * ci : (R)0;
    m[1][0] = qr * dr - qi * di;
    m[1][1] = qr * di + qi * dr;
    const R two = neg ? (R)2 : (R)-2;  // -2 zeta_0 d = two z d
    const R gr = two * (zr * dr - zi * di), gi = two * (zr * di + zi * dr);
    const R d2r = dr * dr - di * di, d2i = (R)2 * dr * di;
#pragma unroll
    for (int p = 1; p < DEG; p++) {
        const R s = (R)1 / (R)(p + 1);
        R tr = (gr * m[p][0] - gi * m[p][1]) * s, ti = (gr * m[p][1] + gi * m[p][0]) * s;
        if (p > 1) {
            const R u = (R)(-2 * (p - 1)) / (R)((p + 1) * p);
            tr += u * (d2r * m[p - 1][0] - d2i * m[p - 1][1]);
            ti += u * (d2r * m[p - 1][1] + d2i * m[p - 1][0]);
        }
        m[p + 1][0] = tr;
        m[p + 1][1] = ti;
    }
}

// Adds A rho^k sq[k - 1] (sum_p m_p k^p) to the column's sums, k = -ROWS/2 ...
// ROWS/2 - 1; u = rho, v = 1 / rho.  Even and odd powers are shared by +k and -k.
template <int ROWS, int DEG, typename R, typename R2>
__device__ inline void add_column(R ar, R ai, R ur, R ui, R vr, R vi, const R (&m)[DEG + 1][2], const R2 *sq,
                                  R (&acc_re)[ROWS], R (&acc_im)[ROWS]) {
    constexpr int H = ROWS / 2, E = DEG / 2 * 2, O = (DEG - 1) / 2 * 2 + 1;
    acc_re[H] += ar * m[0][0] - ai * m[0][1];
    acc_im[H] += ar * m[0][1] + ai * m[0][0];
    R pr = ar, pi = ai, nr = ar, ni = ai;
#pragma unroll
    for (int k = 1; k <= H; k++) {
        const R k1 = (R)k, k2 = (R)(k * k);
        R er = m[E][0], ei = m[E][1], qr = m[O][0], qi = m[O][1];
#pragma unroll
        for (int p = E - 2; p >= 0; p -= 2) {
            er = fma(er, k2, m[p][0]);
            ei = fma(ei, k2, m[p][1]);
        }
#pragma unroll
        for (int p = O - 2; p >= 1; p -= 2) {
            qr = fma(qr, k2, m[p][0]);
            qi = fma(qi, k2, m[p][1]);
        }
        const R2 s = sq[k - 1];
        if (k < H) {
            const R xr = fma(pr, ur, -(pi * ui));
            pi = fma(pr, ui, pi * ur);
            pr = xr;
            const R tr = fma(pr, s.x, -(pi * s.y)), ti = fma(pr, s.y, pi * s.x);
            const R fr = fma(qr, k1, er), fi = fma(qi, k1, ei);
            acc_re[H + k] = fma(tr, fr, fma(-ti, fi, acc_re[H + k]));
            acc_im[H + k] = fma(tr, fi, fma(ti, fr, acc_im[H + k]));
        }
        {
            const R xr = fma(nr, vr, -(ni * vi));
            ni = fma(nr, vi, ni * vr);
            nr = xr;
            const R tr = fma(nr, s.x, -(ni * s.y)), ti = fma(nr, s.y, ni * s.x);
            const R fr = fma(qr, -k1, er), fi = fma(qi, -k1, ei);
            acc_re[H - k] = fma(tr, fr, fma(-ti, fi, acc_re[H - k]));
            acc_im[H - k] = fma(tr, fi, fma(ti, fr, acc_im[H - k]));
        }
    }
}

// ONE: a segment is one tile of kMixedTile beamlets at most, so its FP32 sums
// need no compensation (and 32 rows their registers).
template <int ROWS, int DEG, bool ONE>
__global__ void __launch_bounds__(256) cut_column_mixed_kernel(EvalGeom g, const Rec32 *__restrict__ rec,
                                                               const RecCut32 *__restrict__ cut, FaddeevaCoef fc,
                                                               int32_t seg_base, float4 *__restrict__ partial) {
    constexpr int H = ROWS / 2, WAVES = 4;
    constexpr int kVec4 = offsetof(Rec32, sq) / 16;
    __shared__ float4 tile[kMixedTile][kVec4];
    __shared__ RecCut32 ctile[kMixedTile];
    __shared__ float2 sq[kMixedTile][H];
    const int w = work_item(blockIdx.x, gridDim.x);
    if (w >= g.work) return;
    const int tiles = g.tiles_x * g.tiles_y;
    const int seg = w / tiles;
    const int t = w - seg * tiles;
    const int ty = t / g.tiles_x, tx = t - ty * g.tiles_x;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int ix = tx * 64 + lane;
    const int iy0 = (ty * WAVES + wv) * ROWS;
    const double a = g.a0 + ix * g.dx, bh = g.b0 + (iy0 + H) * g.dy, dy = g.dy;
    const float dyf = (float)dy;
    constexpr float kLog2e = 1.4426950408889634f, kInv2Pi = 0.15915494309189535f;

    constexpr int KS = ONE ? 1 : ROWS;
    float s_re[KS], s_im[KS], c_re[KS], c_im[KS], acc_re[ROWS], acc_im[ROWS];
#pragma unroll
    for (int k = 0; k < ROWS; k++) acc_re[k] = acc_im[k] = 0.0f;
#pragma unroll
    for (int k = 0; k < KS; k++) s_re[k] = s_im[k] = c_re[k] = c_im[k] = 0.0f;
    const int64_t jb = (int64_t)seg * g.seg_len;
    const int64_t je = min(g.n, jb + g.seg_len);
    for (int64_t j0 = jb; j0 < je; j0 += kMixedTile) {
        const int cnt = (int)min((int64_t)kMixedTile, je - j0);
        __syncthreads();
        {
            for (int i = threadIdx.x; i < cnt * kVec4; i += 64 * WAVES) {
                const int j = i / kVec4, k = i - j * kVec4;
                tile[j][k] = reinterpret_cast<const float4 *>(rec + j0 + j)[k];
            }
            const float4 *cs = reinterpret_cast<const float4 *>(cut + j0);
            float4 *cd4 = reinterpret_cast<float4 *>(ctile);
            for (int i = threadIdx.x; i < cnt * 2; i += 64 * WAVES) cd4[i] = cs[i];
            for (int i = threadIdx.x; i < cnt * H; i += 64 * WAVES) {
                const Rec32 &r = rec[j0 + i / H];
                const double2 s = rotor_sigma(r.p[5], (double)r.m[5] / il2_dev(), dy, i % H + 1);
                sq[i / H][i % H] = make_float2((float)s.x, (float)s.y);
            }
        }
        __syncthreads();
        for (int jj = 0; jj < cnt; jj++) {
            const Rec32 &r = *reinterpret_cast<const Rec32 *>(tile[jj]);
            const RecCut32 &c = ctile[jj];
            // anchor row and step, as the rotor form
            const double da = a - r.arho, db = bh - r.brho;
            const double q = r.p[2] + r.p[4] * da;
            const double T0 = r.p[0] + da * (r.p[1] + r.p[3] * da) + db * (q + r.p[5] * db);
            const double T1 = dy * (q + 2.0 * r.p[5] * db);
            const float t1 = (float)(T1 - rint(T1));
            const float daf = (float)da, dbf = (float)db;
            const float qf = r.m[2] + r.m[4] * daf;
            const float L = r.m[0] + daf * (r.m[1] + r.m[3] * daf) + dbf * (qf + r.m[5] * dbf);
            const float U1 = fminf(fmaxf(dyf * (qf + 2.0f * r.m[5] * dbf), -64.0f), 64.0f);
            float zr = fmaf(c.zb[0], dbf, fmaf(c.za[0], daf, c.z0[0]));
            float zi = fmaf(c.zb[1], dbf, fmaf(c.za[1], daf, c.z0[1]));
            const bool neg = zr < 0.0f;
            zr = neg ? -zr : zr;
            zi = neg ? -zi : zi;
            const float2 wz = faddeeva32(fc, -zi, zr);
            const float xr = (zr * zr - zi * zi) * kLog2e, xi = 2.0f * zr * zi * kInv2Pi;  // zeta_0^2
            const bool big = !neg || xr < 0.0f;
            const float La = big ? L - xr : L;
            const float pa = __builtin_amdgcn_fractf((float)__builtin_amdgcn_fract(T0) - (big ? xi : 0.0f));
            const float ma = La < -126.0f ? 0.0f : __builtin_amdgcn_exp2f(La);
            const float mc = __builtin_amdgcn_exp2f(-fabsf(xr)), pc = __builtin_amdgcn_fractf(big ? xi : -xi);
            float m[DEG + 1][2];
            edge_poly<DEG>(zr, zi, neg, big, wz.x, wz.y, mc * __builtin_amdgcn_cosf(pc),
                           mc * __builtin_amdgcn_sinf(pc), c.zb[0] * dyf, c.zb[1] * dyf, m);
            const float mu = __builtin_amdgcn_exp2f(U1), md = __builtin_amdgcn_exp2f(-U1);
            const float c1 = __builtin_amdgcn_cosf(t1), s1 = __builtin_amdgcn_sinf(t1);
            add_column<ROWS, DEG>(ma * __builtin_amdgcn_cosf(pa), ma * __builtin_amdgcn_sinf(pa), mu * c1, mu * s1,
                                  md * c1, -(md * s1), m, sq[jj], acc_re, acc_im);
        }
        if constexpr (!ONE)
#pragma unroll
            for (int k = 0; k < ROWS; k++) {
                kahan(s_re[k], c_re[k], acc_re[k]);
                kahan(s_im[k], c_im[k], acc_im[k]);
                acc_re[k] = acc_im[k] = 0.0f;
            }
    }
    if (ix >= g.nx) return;
    const int64_t M = (int64_t)g.nx * g.ny;
#pragma unroll
    for (int k = 0; k < ROWS; k++) {
        const int iy = iy0 + k;
        if (iy < g.ny)
            partial[(int64_t)(seg_base + seg) * M + (int64_t)iy * g.nx + ix] =
                ONE ? make_float4(acc_re[k], acc_im[k], 0.0f, 0.0f)
                    : make_float4(s_re[ONE ? 0 : k], s_im[ONE ? 0 : k], c_re[ONE ? 0 : k], c_im[ONE ? 0 : k]);
    }
}

template <int ROWS, int DEG>
__global__ void __launch_bounds__(256) cut_column_fp64_kernel(EvalGeom g, const Rec64 *__restrict__ rec,
                                                              const RecCut64 *__restrict__ cut, FaddeevaCoef fc,
                                                              int32_t seg_base, double2 *__restrict__ partial) {
    constexpr int H = ROWS / 2, WAVES = 4, CH = 64;
    __shared__ Rec64 tile[CH];
    __shared__ RecCut64 ctile[CH];
    __shared__ double2 sq[CH][H];
    const int w = work_item(blockIdx.x, gridDim.x);
    if (w >= g.work) return;
    const int tiles = g.tiles_x * g.tiles_y;
    const int seg = w / tiles;
    const int t = w - seg * tiles;
    const int ty = t / g.tiles_x, tx = t - ty * g.tiles_x;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int ix = tx * 64 + lane;
    const int iy0 = (ty * WAVES + wv) * ROWS;
    const double a = g.a0 + ix * g.dx, bh = g.b0 + (iy0 + H) * g.dy, dy = g.dy;

    double acc_re[ROWS], acc_im[ROWS];
#pragma unroll
    for (int k = 0; k < ROWS; k++) acc_re[k] = acc_im[k] = 0.0;
    const int64_t jb = (int64_t)seg * g.seg_len;
    const int64_t je = min(g.n, jb + g.seg_len);
    for (int64_t j0 = jb; j0 < je; j0 += CH) {
        const int cnt = (int)min((int64_t)CH, je - j0);
        __syncthreads();
        {
            const double2 *src = reinterpret_cast<const double2 *>(rec + j0);
            double2 *dst = reinterpret_cast<double2 *>(tile);
            for (int i = threadIdx.x; i < cnt * 8; i += 64 * WAVES) dst[i] = src[i];
            const double2 *cs = reinterpret_cast<const double2 *>(cut + j0);
            double2 *cd2 = reinterpret_cast<double2 *>(ctile);
            for (int i = threadIdx.x; i < cnt * 4; i += 64 * WAVES) cd2[i] = cs[i];
            for (int i = threadIdx.x; i < cnt * H; i += 64 * WAVES) {
                const Rec64 &r = rec[j0 + i / H];
                sq[i / H][i % H] = rotor_sigma(r.p[5], r.l[5], dy, i % H + 1);
            }
        }
        __syncthreads();
        for (int jj = 0; jj < cnt; jj++) {
            const Rec64 &r = tile[jj];
            const RecCut64 &c = ctile[jj];
            const double da = a - r.arho, db = bh - r.brho;
            const double q = r.p[2] + r.p[4] * da, ql = r.l[2] + r.l[4] * da;
            const double T0 = r.p[0] + da * (r.p[1] + r.p[3] * da) + db * (q + r.p[5] * db);
            const double T1 = dy * (q + 2.0 * r.p[5] * db);
            const double L = r.l[0] + da * (r.l[1] + r.l[3] * da) + db * (ql + r.l[5] * db);
            const double U1 = fmin(fmax(dy * (ql + 2.0 * r.l[5] * db), -44.0), 44.0);
            double zr = c.z0[0] + c.za[0] * da + c.zb[0] * db;
            double zi = c.z0[1] + c.za[1] * da + c.zb[1] * db;
            const bool neg = zr < 0.0;
            zr = neg ? -zr : zr;
            zi = neg ? -zi : zi;
            const cd wz = faddeeva64(fc, -zi, zr);
            const double xr = zr * zr - zi * zi, xi = zr * zi / kPi;  // zeta_0^2, its phase in turns
            const bool big = !neg || xr < 0.0;
            double pa = T0 - rint(T0) - (big ? xi : 0.0), pc = big ? xi : -xi;
            pa -= rint(pa);
            pc -= rint(pc);
            double sa, ca, sc, cc, s1, c1;
            sincospi(2.0 * pa, &sa, &ca);
            sincospi(2.0 * pc, &sc, &cc);
            sincospi(2.0 * (T1 - rint(T1)), &s1, &c1);
            const double ma = exp(big ? L - xr : L), mc = exp(-fabs(xr));
            double m[DEG + 1][2];
            edge_poly<DEG>(zr, zi, neg, big, wz.re, wz.im, mc * cc, mc * sc, c.zb[0] * dy, c.zb[1] * dy, m);
            const double mu = exp(U1), md = exp(-U1);
            add_column<ROWS, DEG>(ma * ca, ma * sa, mu * c1, mu * s1, md * c1, -(md * s1), m, sq[jj], acc_re, acc_im);
        }
    }
    if (ix >= g.nx) return;
    const int64_t M = (int64_t)g.nx * g.ny;
#pragma unroll
    for (int k = 0; k < ROWS; k++) {
        const int iy = iy0 + k;
        if (iy < g.ny)
            partial[(int64_t)(seg_base + seg) * M + (int64_t)iy * g.nx + ix] = make_double2(acc_re[k], acc_im[k]);
    }
}

}  // namespace

hipError_t launch_eval_cut(int precision, int level, const EvalGeom &g, const void *rec, const void *cut,
                           const FaddeevaCoef &fc, int32_t seg_base, void *partial, hipStream_t s) {
    const int grid = (g.work + 7) / 8 * 8;
    if (level == 4 && (precision != 1 || g.seg_len > kMixedTile)) return hipErrorInvalidValue;
    if (precision == 1) {
        auto *r = static_cast<const Rec32 *>(rec);
        auto *c = static_cast<const RecCut32 *>(cut);
        auto *p = static_cast<float4 *>(partial);
        if (level == 4)
            cut_column_mixed_kernel<2 * kCutRows, 5, true><<<grid, 256, 0, s>>>(g, r, c, fc, seg_base, p);
        else if (level == 3)
            cut_column_mixed_kernel<kCutRows, 5, false><<<grid, 256, 0, s>>>(g, r, c, fc, seg_base, p);
        else if (level == 2)
            cut_column_mixed_kernel<kCutRows, 9, false><<<grid, 256, 0, s>>>(g, r, c, fc, seg_base, p);
        else if (level == 1)
            cut_column_mixed_kernel<kCutRows / 2, 9, false><<<grid, 256, 0, s>>>(g, r, c, fc, seg_base, p);
        else
            eval_cut_mixed_kernel<kCutRows32, 4><<<grid, 256, 0, s>>>(g, r, c, fc, seg_base, p);
    } else {
        auto *r = static_cast<const Rec64 *>(rec);
        auto *c = static_cast<const RecCut64 *>(cut);
        auto *p = static_cast<double2 *>(partial);
        if (level == 3)
            cut_column_fp64_kernel<kCutRows, 9><<<grid, 256, 0, s>>>(g, r, c, fc, seg_base, p);
        else if (level == 2)
            cut_column_fp64_kernel<kCutRows, 15><<<grid, 256, 0, s>>>(g, r, c, fc, seg_base, p);
        else if (level == 1)
            cut_column_fp64_kernel<kCutRows / 2, 15><<<grid, 256, 0, s>>>(g, r, c, fc, seg_base, p);
        else
            eval_cut_fp64_kernel<kCutRows64, 4><<<grid, 256, 0, s>>>(g, r, c, fc, seg_base, p);
    }
    return hipGetLastError();
}

}  // namespace gbd
