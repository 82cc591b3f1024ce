// Core of the matrix form for beamlets with weak cross terms (see
// gbd_cross.hip for the method): the FP16 MFMA accumulation of one
// workgroup's 128 x 128 pixel tile over a range of beamlets.
#pragma once

#include "gbd_sep_core.h"

namespace gbd {
namespace cross {

using namespace sep;

constexpr int kWX = 2, kWY = 4;  // wavefronts per workgroup along x and y
constexpr int kBX = 4, kBY = 2;  // 16-pixel blocks per wavefront along x and y
constexpr int kThreads = 64 * kWX * kWY;
static_assert(kCrossTile == 128 && kWX * kWY == 8, "a wavefront forms the factors of two beamlets over twice 64 pixels");
static_assert(16 * kWX * kBX == kCrossTile && 16 * kWY * kBY == kCrossTile, "cross form: host and kernel tiles");

// Scales: |U| <= 2^kUExp and |V| <= 2^kVExp by the setup's bounds, up to the
// factor 2 (U) and 4 (V) that the cross term's share in them can add
// (FLAG_CROSS2 bounds it); FP16 holds 65504.
constexpr int kUExp = 13, kVExp = 12;

// Words of a U and a V factor in LDS:
//   LEVEL 1: U_h, U_l, (xu U)_h            A_h, A_l, W_h, W_l
//   LEVEL 2: ... and (xu U)_l, (xu)^2/2 U_h   A_h, A_l, (vA)_h, (vA)_l
// with A = (Vr, -Vi), W = (Vi, Vr) its quarter turn.
template <int LEVEL>
struct CrossCfg {
    static constexpr int NU = LEVEL == 1 ? 3 : 5, NV = 4;
};
// A Rec32 up to the rotor tables, uniform over the wavefront: scalar loads.
typedef uint32_t u16w __attribute__((ext_vector_type(16), aligned(16)));
typedef uint32_t u8w __attribute__((ext_vector_type(8), aligned(16)));
typedef uint32_t u4w __attribute__((ext_vector_type(4), aligned(16)));
struct CrossRec {
    u16w a;
    u8w b;
    u4w c;
    __device__ uint32_t word(int k) const { return k < 16 ? a[k & 15] : k < 24 ? b[k & 7] : c[k & 3]; }
    __device__ double f64(int k) const {
        return __builtin_bit_cast(double, (uint64_t)word(k) | ((uint64_t)word(k + 1) << 32));
    }
    __device__ float f32(int k) const { return __builtin_bit_cast(float, word(k)); }
};
__device__ inline CrossRec cross_rec(const Rec32 *__restrict__ r) {
    CrossRec w;
    w.a = *reinterpret_cast<const u16w *>(r);
    w.b = *(reinterpret_cast<const u8w *>(r) + 2);
    w.c = *(reinterpret_cast<const u4w *>(r) + 6);
    return w;
}
static_assert(offsetof(Rec32, sq) == 112 && offsetof(Rec32, m) == 64 && offsetof(Rec32, pad) == 108, "Rec32 layout");

template <int LEVEL>
struct alignas(16) CrossLds {
    // [buffer][range][block][part][pixel in block][beamlet in pass, swizzled as SepHLdsT]
    uint32_t lu[2][kWX][kBX][CrossCfg<LEVEL>::NU][16][16];
    uint32_t lv[2][kWY][kBY][CrossCfg<LEVEL>::NV][16][16];
};
static_assert(sizeof(CrossLds<2>) <= 163840, "a workgroup's 160 KiB of LDS");

__device__ inline h8 pk_scale(h8 a, h2 s) {
    h8 r;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const h2 x = h2{a[2 * i], a[2 * i + 1]} * s;
        r[2 * i] = x[0];
        r[2 * i + 1] = x[1];
    }
    return r;
}
// rot_halves of each packed pair
__device__ inline h8 rot8(h8 a) {
    uint4 v = __builtin_bit_cast(uint4, a);
    v.x = rot_halves(v.x);
    v.y = rot_halves(v.y);
    v.z = rot_halves(v.z);
    v.w = rot_halves(v.w);
    return __builtin_bit_cast(h8, v);
}

// As sep_accumulate_h: passes of 16 beamlets, factors formed one pass ahead
// between the products.  A wavefront forms all factors of two beamlets, so
// that a beamlet's record is uniform (scalar loads, half a pass ahead) and two
// neighbouring words of a pixel leave in one LDS store; with four beamlets to
// a wavefront, records read from LDS by every lane and single words stored,
// LDS took half of a pass (the kernel on 12,892 beamlets and 1024 x 1024
// pixels 580 -> 516 us in a profiled run).  With (u, v)
// the pixel's offset from the tile's centre in half tiles and x = the
// beamlet's cross coefficient times a half tile squared, the factors carry
// the cross term along the centre's row and column and
//   e^(x u v) = 1 + (xu) v                      (LEVEL 1, |x| <= 2^-10)
//             = 1 + (xu) v + (xu)^2/2 v^2       (LEVEL 2, |x| <= 2^-6)
// the rest of it, as further products into the same sums.  The leading
// product takes hi hi + hi lo + lo hi; the small ones hi hi where that keeps
// them to 1e-7 of a term (LEVEL 1's first, LEVEL 2's second), else all three.
template <int LEVEL>
__device__ inline void cross_accumulate(const SepGeom &g, const Rec32 *__restrict__ rec, int64_t jb, int64_t je, int tx,
                                        int ty, float P, CrossLds<LEVEL> &L, f4 (&accR)[kBY][kBX],
                                        f4 (&accI)[kBY][kBX]) {
    constexpr int NU = CrossCfg<LEVEL>::NU, NV = CrossCfg<LEVEL>::NV;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wx = wv % kWX, wy = wv / kWX;
    const int X0 = tx * kCrossTile, Y0 = ty * kCrossTile;
    const int li = lane & 15, lk = lane >> 4, sw = swz(li);
    auto &lu = L.lu;
    auto &lv = L.lv;
    constexpr double half = 0.5 * kCrossTile;
    const double ac = g.a0 + (X0 + half - 0.5) * g.dx, bc = g.b0 + (Y0 + half - 0.5) * g.dy;
    // this lane's two columns and rows, as factors; their u and v
    double ax[2], by[2];
    float u[2];
#pragma unroll
    for (int h = 0; h < 2; h++) {
        ax[h] = g.a0 + (X0 + 64 * h + lane) * g.dx;
        by[h] = g.b0 + (Y0 + 64 * h + lane) * g.dy;
        u[h] = (float)((64 * h + lane + 0.5 - half) / half);
    }
    const float xs_re = (float)(0.69314718055994531 * half * half * g.dx * g.dy);  // per log2 unit
    const double xs_im = 2.0 * kPi * half * half * g.dx * g.dy;                    // per turn
    // the v of the rows that this lane reads as operands
    h2 vr_[kBY];
#pragma unroll
    for (int p = 0; p < kBY; p++) {
        const _Float16 h = (_Float16)(float)((16 * (wy * kBY + p) + li + 0.5 - half) / half);
        vr_[p] = h2{h, h};
    }
    const Rec32 *__restrict__ srec = rec + jb;
    const int n = (int)(je - jb);
    // beamlet `which` of this wavefront's two in the pass at i0 (past the end:
    // the last one's record, of amplitude zero)
    auto record = [&](int i0, int which) { return cross_rec(srec + min(i0 + 2 * wv + which, n - 1)); };
    auto live = [&](int i0, int which) { return i0 + 2 * wv + which < n; };
    auto form_u = [&](const CrossRec &r, bool in, uint32_t (&o)[2][NU]) {
        const double arho = r.f64(0), dbc = bc - r.f64(2), p4 = r.f64(12);
        const float m4 = r.f32(20), ub = r.f32(27), dbcf = (float)dbc, m0 = in ? r.f32(16) : -INFINITY;
        const double c1 = r.f64(6) + p4 * dbc;
        const float l1 = r.f32(17) + m4 * dbcf;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            float re, im;
            // exponents near zero, so that their rounding stays below the phase's;
            // the range's powers of two multiplied in afterwards
            const double da = ax[h] - arho;  // (offsets rounded once, from FP64)
            factor(da, (float)da, r.f64(4), c1, r.f64(10), m0 - ub, l1, r.f32(19), re, im);
            re *= (float)(1 << kUExp);
            im *= (float)(1 << kUExp);
            split_halves(re, im, o[h][0], o[h][1]);
            const float xr = m4 * (xs_re * u[h]), xi = (float)(p4 * (xs_im * (double)u[h]));
            const float r1 = xr * re - xi * im, i1 = xr * im + xi * re;
            if constexpr (LEVEL == 1) {
                o[h][2] = __builtin_bit_cast(uint32_t, h2{(_Float16)r1, (_Float16)i1});
            } else {
                split_halves(r1, i1, o[h][2], o[h][3]);
                const float r2 = 0.5f * (xr * r1 - xi * i1), i2 = 0.5f * (xr * i1 + xi * r1);
                o[h][4] = __builtin_bit_cast(uint32_t, h2{(_Float16)r2, (_Float16)i2});
            }
        }
    };
    auto form_v = [&](const CrossRec &r, uint32_t (&o)[2][NV]) {
        const double dac = ac - r.f64(0), brho = r.f64(2), dbc = bc - brho, pa = r.f64(12) * dac;
        const float m4 = r.f32(20), dacf = (float)dac, dbcf = (float)dbc;
        const double c0 = -pa * dbc, c1 = r.f64(8) + pa;
        const float l0 = r.f32(27) - P - m4 * dacf * dbcf, l1 = r.f32(18) + m4 * dacf;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            float re, im;
            const double db = by[h] - brho;
            factor(db, (float)db, c0, c1, r.f64(14), l0, l1, r.f32(21), re, im);
            re *= (float)(1 << kVExp);
            im *= (float)(1 << kVExp);
            split_halves_conj(re, im, o[h][0], o[h][1]);
            if constexpr (LEVEL == 1) {
                o[h][2] = rot_halves(o[h][0]);
                o[h][3] = rot_halves(o[h][1]);
            } else {
                split_halves_conj(u[h] * re, u[h] * im, o[h][2], o[h][3]);
            }
        }
    };
    // both beamlets' words of each pixel in one store
    const int col = 4 * ((wv >> 1) ^ sw) + 2 * (wv & 1);
    auto put = [](uint32_t *dst, uint32_t a, uint32_t b) { *reinterpret_cast<uint2 *>(dst) = make_uint2(a, b); };
    auto store_u = [&](int buf, const uint32_t (&a)[2][NU], const uint32_t (&b)[2][NU]) {
#pragma unroll
        for (int h = 0; h < 2; h++)
#pragma unroll
            for (int k = 0; k < NU; k++) put(&lu[buf][h][lk][k][li][col], a[h][k], b[h][k]);
    };
    auto store_v = [&](int buf, const uint32_t (&a)[2][NV], const uint32_t (&b)[2][NV]) {
#pragma unroll
        for (int h = 0; h < 2; h++)
#pragma unroll
            for (int k = 0; k < NV; k++) put(&lv[buf][2 * h + (lane >> 5)][lk & 1][k][li][col], a[h][k], b[h][k]);
    };
#pragma unroll
    for (int p = 0; p < kBY; p++)
#pragma unroll
        for (int q = 0; q < kBX; q++) accR[p][q] = accI[p][q] = f4{0.0f, 0.0f, 0.0f, 0.0f};

    uint32_t ua[2][NU], ub[2][NU], va[2][NV], vb[2][NV];
    CrossRec ra = record(0, 0), rb = record(0, 1);
    form_u(ra, live(0, 0), ua);
    form_v(ra, va);
    form_u(rb, live(0, 1), ub);
    form_v(rb, vb);
    store_u(0, ua, ub);
    store_v(0, va, vb);
    ra = record(16, 0);
    rb = record(16, 1);
    __syncthreads();
    const int rd = 4 * (lk ^ sw);  // this lane's operand group in a row
    int buf = 0;
    for (int i0 = 0; i0 < n; i0 += 16) {
        h8 b[kBX][NU];
#pragma unroll
        for (int q = 0; q < kBX; q++)
#pragma unroll
            for (int k = 0; k < NU; k++) b[q][k] = operand(&lu[buf][wx][q][k][li][rd]);
        h8 a[NV], w[NV], a2, w2;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            // operands first: a load cannot pass the factors' stores to LDS
            static_assert(kBX % 2 == 0, "two blocks of one row at a time");
            if (2 * k % kBX == 0) {
                const int p = 2 * k / kBX;
#pragma unroll
                for (int t = 0; t < NV; t++) a[t] = operand(&lv[buf][wy][p][t][li][rd]);
                if constexpr (LEVEL == 1) {
                    w[0] = a[2];
                    w[1] = a[3];
                    a2 = pk_scale(a[0], vr_[p]);
                    w2 = pk_scale(w[0], vr_[p]);
                } else {
#pragma unroll
                    for (int t = 0; t < NV; t++) w[t] = rot8(a[t]);
                    a2 = pk_scale(a[2], vr_[p]);
                    w2 = pk_scale(w[2], vr_[p]);
                }
            }
            // the next pass's factors, a quarter to a section
            if (k == 0) form_u(ra, live(i0 + 16, 0), ua);
            if (k == 1) {
                form_v(ra, va);
                ra = record(i0 + 32, 0);
            }
            if (k == 2) {
                form_u(rb, live(i0 + 16, 1), ub);
                store_u(buf ^ 1, ua, ub);
            }
            if (k == 3) {
                form_v(rb, vb);
                store_v(buf ^ 1, va, vb);
                rb = record(i0 + 32, 1);
            }
#pragma unroll
            for (int i = 0; i < 2; i++) {
                const int m = 2 * k + i, p = m / kBX, q = m % kBX;
                auto mac = [&](const h8 &x, const h8 &y, f4 &c) {
                    c = __builtin_amdgcn_mfma_f32_16x16x32_f16(x, y, c, 0, 0, 0);
                };
                f4 &R = accR[p][q], &I = accI[p][q];
                mac(a[0], b[q][0], R);
                mac(w[0], b[q][0], I);
                mac(a[0], b[q][1], R);
                mac(w[0], b[q][1], I);
                mac(a[1], b[q][0], R);
                mac(w[1], b[q][0], I);
                if constexpr (LEVEL == 1) {
                    mac(a2, b[q][2], R);
                    mac(w2, b[q][2], I);
                } else {
                    mac(a[2], b[q][2], R);
                    mac(w[2], b[q][2], I);
                    mac(a[2], b[q][3], R);
                    mac(w[2], b[q][3], I);
                    mac(a[3], b[q][2], R);
                    mac(w[3], b[q][2], I);
                    mac(a2, b[q][4], R);
                    mac(w2, b[q][4], I);
                }
            }
            if constexpr (LEVEL == 1) {
                // four VALU instructions behind each MFMA, section by section:
                // left to itself the scheduler forms half of the factors
                // before any product (LEVEL 2 has no registers left for it)
#pragma unroll
                for (int i = 0; i < 16; i++) {
                    __builtin_amdgcn_sched_group_barrier(0x2, 4, 0);
                    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();
        buf ^= 1;
    }
}

}  // namespace cross
}  // namespace gbd
