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
static_assert(kBX % kWY == 0 && kBY % kWX == 0, "a lane forms one U and one V factor per quad of beamlets");
static_assert(16 * kWX * kBX == kCrossTile && 16 * kWY * kBY == kCrossTile, "cross form: host and kernel tiles");

// Scales: |U| <= 2^kUExp and |V| <= 2^kVExp by the setup's bounds, up to the
// factor 2 (U) and 4 (V) that the cross term's share in them can add
// (kCrossShift); FP16 holds 65504.
constexpr int kUExp = 13, kVExp = 12;

// Words of a U and a V factor in LDS:
//   LEVEL 1: U_h, U_l, (xu U)_h            A_h, A_l, W_h, W_l
//   LEVEL 2: ... and (xu U)_l, (xu)^2/2 U_h   A_h, A_l, (vA)_h, (vA)_l
// with A = (Vr, -Vi), W = (Vi, Vr) its quarter turn.
template <int LEVEL>
struct CrossCfg {
    static constexpr int NU = LEVEL == 1 ? 3 : 5, NV = 4;
};
constexpr int kRecWords = 28;  // the words of a Rec32 before the rotor tables
static_assert(offsetof(Rec32, sq) == 4 * kRecWords, "Rec32 layout");
constexpr int kWordM0 = offsetof(Rec32, m) / 4, kWordU = offsetof(Rec32, pad) / 4;

template <int LEVEL>
struct alignas(16) CrossLds {
    // [buffer][range][block][part][pixel in block][beamlet in pass, swizzled as SepHLdsT]
    uint32_t lu[2][kWX][kBX][CrossCfg<LEVEL>::NU][16][16];
    uint32_t lv[2][kWY][kBY][CrossCfg<LEVEL>::NV][16][16];
    // [buffer][beamlet in pass][word]; the rows past 16 take the idle threads' words
    uint32_t rs[2][(kThreads + kRecWords - 1) / kRecWords][kRecWords];
};
static_assert(sizeof(CrossLds<2>) <= 163840, "a workgroup's 160 KiB of LDS");
static_assert(kThreads >= 16 * kRecWords, "one word per thread and pass");

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

// As sep_accumulate_h (passes of 16 beamlets, records staged two passes
// ahead, factors formed one pass ahead between the products).  With (u, v)
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
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int wx = wv % kWX, wy = wv / kWX;
    const int X0 = tx * kCrossTile, Y0 = ty * kCrossTile;
    const int li = lane & 15, lk = lane >> 4, sw = swz(li);
    auto &lu = L.lu;
    auto &lv = L.lv;
    auto &rs = L.rs;
    // this wavefront forms U block wy of x range wx and V block wx of y range wy
    const int ix = X0 + 16 * (wx * kBX + wy) + li, iy = Y0 + 16 * (wy * kBY + wx) + li;
    constexpr double half = 0.5 * kCrossTile;
    const double ac = g.a0 + (X0 + half - 0.5) * g.dx, bc = g.b0 + (Y0 + half - 0.5) * g.dy;
    const double ax = g.a0 + ix * g.dx, by = g.b0 + iy * g.dy;
    const float u = (float)((ix - X0 + 0.5 - half) / half), v = (float)((iy - Y0 + 0.5 - half) / half);
    const float xs_re = (float)(0.69314718055994531 * half * half * g.dx * g.dy) * u;  // per log2 unit, times u
    const double xs_im = 2.0 * kPi * half * half * g.dx * g.dy * (double)u;            // per turn, times u
    // the v of the rows that this lane reads as operands
    h2 vr_[kBY];
#pragma unroll
    for (int p = 0; p < kBY; p++) {
        const _Float16 h = (_Float16)(float)((16 * (wy * kBY + p) + li + 0.5 - half) / half);
        vr_[p] = h2{h, h};
    }
    const Rec32 *__restrict__ srec = rec + jb;
    const int n = (int)(je - jb);
    const int st = threadIdx.x, sr = st / kRecWords, sc = st - sr * kRecWords;
    const uint32_t pad_w = sc == kWordM0 ? 0xff800000u : sc == kWordU ? kPadU : 0u;
    auto stage_load = [&](int i0) {
        const int i = i0 + sr;
        const uint32_t w = reinterpret_cast<const uint32_t *>(srec + (i < n ? i : 0))[sc];
        const uint32_t keep = 0u - (uint32_t)(i < n);
        return (w & keep) | (pad_w & ~keep);
    };
    auto publish = [&](int sbuf, int buf, int qd) {
        const uint32_t *r = rs[sbuf][4 * qd + lk];
        uint4 w[7];
#pragma unroll
        for (int k = 0; k < 7; k++) w[k] = reinterpret_cast<const uint4 *>(r)[k];
        auto f64 = [&](int k) {
            const uint4 &q = w[k >> 2];
            const uint32_t lo = (k & 3) == 0 ? q.x : q.z, hi = (k & 3) == 0 ? q.y : q.w;
            return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
        };
        auto f32 = [&](int k) {
            const uint4 &q = w[k >> 2];
            const uint32_t x = (k & 3) == 0 ? q.x : (k & 3) == 1 ? q.y : (k & 3) == 2 ? q.z : q.w;
            return __builtin_bit_cast(float, x);
        };
        const double arho = f64(0), brho = f64(2), p4 = f64(12);
        const float m4 = f32(20), ub = f32(27);
        const double dac = ac - arho, dbc = bc - brho, pa = p4 * dac;
        const float dacf = (float)dac, dbcf = (float)dbc;
        const int col = 4 * (qd ^ sw) + lk;
        float re, im;
        uint32_t hi, lo;
        // exponents near zero, so that their rounding stays below the phase's;
        // the range's powers of two multiplied in afterwards
        const double da = ax - arho, db = by - brho;  // (offsets rounded once, from FP64)
        factor(da, (float)da, f64(4), f64(6) + p4 * dbc, f64(10), f32(16) - ub, f32(17) + m4 * dbcf, f32(19), re,
               im);
        re *= (float)(1 << kUExp);
        im *= (float)(1 << kUExp);
        split_halves(re, im, hi, lo);
        lu[buf][wx][wy][0][li][col] = hi;
        lu[buf][wx][wy][1][li][col] = lo;
        const float xr = m4 * xs_re, xi = (float)(p4 * xs_im);
        float r1 = xr * re - xi * im, i1 = xr * im + xi * re;
        if constexpr (LEVEL == 1) {
            lu[buf][wx][wy][2][li][col] = __builtin_bit_cast(uint32_t, h2{(_Float16)r1, (_Float16)i1});
        } else {
            split_halves(r1, i1, hi, lo);
            lu[buf][wx][wy][2][li][col] = hi;
            lu[buf][wx][wy][3][li][col] = lo;
            const float r2 = 0.5f * (xr * r1 - xi * i1), i2 = 0.5f * (xr * i1 + xi * r1);
            lu[buf][wx][wy][4][li][col] = __builtin_bit_cast(uint32_t, h2{(_Float16)r2, (_Float16)i2});
        }
        factor(db, (float)db, -pa * dbc, f64(8) + pa, f64(14), ub - P - m4 * dacf * dbcf, f32(18) + m4 * dacf,
               f32(21), re, im);
        re *= (float)(1 << kVExp);
        im *= (float)(1 << kVExp);
        split_halves_conj(re, im, hi, lo);
        lv[buf][wy][wx][0][li][col] = hi;
        lv[buf][wy][wx][1][li][col] = lo;
        if constexpr (LEVEL == 1) {
            lv[buf][wy][wx][2][li][col] = rot_halves(hi);
            lv[buf][wy][wx][3][li][col] = rot_halves(lo);
        } else {
            split_halves_conj(v * re, v * im, hi, lo);
            lv[buf][wy][wx][2][li][col] = hi;
            lv[buf][wy][wx][3][li][col] = lo;
        }
    };
#pragma unroll
    for (int p = 0; p < kBY; p++)
#pragma unroll
        for (int q = 0; q < kBX; q++) accR[p][q] = accI[p][q] = f4{0.0f, 0.0f, 0.0f, 0.0f};

    {
        const uint32_t w0 = stage_load(0), w1 = stage_load(16);
        rs[0][sr][sc] = w0;
        rs[1][sr][sc] = w1;
    }
    __syncthreads();
#pragma unroll
    for (int qd = 0; qd < 4; qd++) publish(0, 0, qd);
    __syncthreads();
    const int rd = 4 * (lk ^ sw);  // this lane's operand group in a row
    int buf = 0;
    for (int i0 = 0; i0 < n; i0 += 16) {
        const uint32_t wnext = stage_load(i0 + 32);
        __builtin_amdgcn_sched_barrier(0);  // the load stays a pass ahead of its use
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
            publish(buf ^ 1, buf ^ 1, k);
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
        rs[buf][sr][sc] = wnext;
        __syncthreads();
        buf ^= 1;
    }
}

}  // namespace cross
}  // namespace gbd
