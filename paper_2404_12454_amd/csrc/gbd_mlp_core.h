// Device functions shared by the surrogate network's kernels.
#pragma once

#include "gbd_internal.h"

#include <math.h>

#include <type_traits>

namespace gbd {
namespace mlp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ inline float sigmoid(float z) { return 1.0f / (1.0f + expf(-z)); }
__device__ inline float silu(float z) { return z * sigmoid(z); }
__device__ inline float dsilu(float z) {
    const float s = sigmoid(z);
    return s * (1.0f + z * (1.0f - s));
}

// Layer l's weight W[o][k] in BF16 to its places as an operand of the forward
// product (column o, K index k) and of the back-propagated one (column k, K index o)
__device__ inline void pack_weight(const MlpNet &n, int l, int o, int k, float v) {
    const int steps = mlp_pack_tiles(n.W) / 2;
    const int64_t at = l * mlp_pack_layer(n.W);
    const uint16_t b = __builtin_bit_cast(uint16_t, (__bf16)v);
    auto place = [&](int c, int q) { return ((c >> 4) * steps + (q >> 5)) * 512 + ((c & 15) + 16 * (q >> 3 & 3)) * 8 + (q & 7); };
    n.wf[at + place(o, k)] = b;
    if (l > 0) n.wb[at + place(k, o)] = b;
}
// the same for flat parameter i, if it is a hidden layer's weight
__device__ inline void pack_param(const MlpNet &n, int64_t i, float v) {
    for (int l = 0; l < n.D; l++)
        if (i >= n.woff[l] && i < n.boff[l]) {
            const int fan = l == 0 ? n.n_in : n.W, j = (int)(i - n.woff[l]);
            pack_weight(n, l, j / fan, j % fan, v);
        }
}

__device__ inline void adamw_step(float &p, float g, float &m, float &v, float lr, float b1, float b2, float eps, float wd,
                                  float c1, float c2) {
    const float mi = b1 * m + (1.0f - b1) * g;
    const float vi = b2 * v + (1.0f - b2) * g * g;
    m = mi;
    v = vi;
    const float mh = mi / c1, vh = vi / c2;
    p = p - lr * (mh / (sqrtf(vh) + eps) + wd * p);
}

// Column sums over a batch, in parallel and in a fixed order: a block of
// 256 threads takes 32 columns, thread (c, r) sums rows r, r + 8, ... of
// column c (coalesced across c), and the 8 partial sums of a column are
// added in order r = 0 ... 7.  out(i, sum_b wgt[b] X[b][i]) for i < W (wgt
// null: weight 1), and with bias_col also out(W, sum_b wgt[b]).
constexpr int kSumCols = 32, kSumRows = 8;
template <class F>
__device__ inline void column_sums(const float *__restrict__ X, const float *__restrict__ wgt, int B, int W,
                                   bool bias_col, int block, F out) {
    __shared__ float part[kSumRows][kSumCols];
    const int c = threadIdx.x % kSumCols, r = threadIdx.x / kSumCols;
    const int i = block * kSumCols + c;
    float acc = 0.0f;
    if (i < W) {
        // 16 rows' loads under way at once, then 4 (100 rows: 12.5 a thread)
        int b = r;
        auto rows = [&](auto count) {
            constexpr int N = decltype(count)::value;
            for (; b + (N - 1) * kSumRows < B; b += N * kSumRows) {
                float x[N], w[N];
#pragma unroll
                for (int k = 0; k < N; k++) {
                    x[k] = X[(int64_t)(b + k * kSumRows) * W + i];
                    w[k] = wgt ? wgt[b + k * kSumRows] : 1.0f;
                }
#pragma unroll
                for (int k = 0; k < N; k++) acc = fmaf(w[k], x[k], acc);
            }
        };
        rows(std::integral_constant<int, 16>());
        rows(std::integral_constant<int, 4>());
        rows(std::integral_constant<int, 1>());
    } else if (bias_col && i == W) {
        for (int b = r; b < B; b += kSumRows) acc += wgt ? wgt[b] : 1.0f;
    }
    part[r][c] = acc;
    __syncthreads();
    if (r == 0 && (i < W || (bias_col && i == W))) {
        float s = part[0][c];
#pragma unroll
        for (int k = 1; k < kSumRows; k++) s += part[k][c];
        out(i, s);
    }
}

}  // namespace mlp
}  // namespace gbd
