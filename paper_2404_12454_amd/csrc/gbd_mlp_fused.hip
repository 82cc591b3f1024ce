// The surrogate network in BF16 mode by two kernels instead of one per
// operation: a training step of the 5-128-128-128-1 network on 256 rows was
// about 20 launches of 2 ... 10 us each, bound by launch and load latency and
// not by its 50 MFLOP (101 us a step; now 17.8, the two kernels 16.5 of them).
// A row's activations, forward and back-propagated, need no other row, so
// mlp_rows_kernel keeps 16 rows (one MFMA tile) per workgroup in LDS and
// registers through all layers and back; the gradients, which sum over the
// rows, then take one kernel for all layers, with the optimiser's step behind
// each one.
#include "gbd_mlp_core.h"

namespace gbd {

namespace {

using namespace mlp;

typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint16_t shortx4 __attribute__((ext_vector_type(4)));

constexpr int kRows = 16;               // rows per workgroup
constexpr int kRowWaves = 8;            // wavefront w takes the column tiles w, w + 8

__device__ inline uint16_t bf(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }

// The operands of one wavefront's column tile, K steps of 32, as packed: one
// kilobyte a load, half the bytes of the FP32 weights, which 16 workgroups
// each fetch whole, and nothing to convert or mask.
template <int S>
struct Weights {
    uint4 v[S];
    __device__ void load(const uint16_t *__restrict__ layer, int tile, int lane, int K) {
        const uint4 *p = reinterpret_cast<const uint4 *>(layer) + (int64_t)tile * S * 64 + lane;
#pragma unroll
        for (int s = 0; s < S; s++) v[s] = 32 * s < K ? p[64 * s] : make_uint4(0u, 0u, 0u, 0u);  // uniform
    }
};

// Four K ranges' partial products, added in their order: with K <= 128 one
// step of 32 each, else two (K <= 256); a step past K adds zeros.
template <int S>
__device__ inline floatx4 product(const Weights<S> &b, const uint16_t *__restrict__ a, int K, int kg) {
    const int ks = S > 4 && K > 128 ? 2 : 1;
    floatx4 p[4];
#pragma unroll
    for (int w = 0; w < 4; w++) p[w] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < S; s++) {
        const bf16x8 x = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(a + 32 * s + 8 * kg));
        const bf16x8 y = __builtin_bit_cast(bf16x8, b.v[s]);
        if (ks == 2)  // steps 0, 1 | 2, 3 | ...
            p[s / 2 & 3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, p[s / 2 & 3], 0, 0, 0);
        else if (s < 4)
            p[s & 3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, p[s & 3], 0, 0, 0);
    }
    return ((p[0] + p[1]) + p[2]) + p[3];
}

// Forward pass (and with BWD the back-propagated dZ) of the rows
// 16 blockIdx ... + 15: T column tiles of 16 per wavefront (W <= 128 T).  Lane
// l of a product's result holds rows 4 (l / 16) + e and column l % 16 of its
// tile, forward and backward alike.  The kernel is a chain of short products
// on a handful of CUs, so what it costs is latency: with T = 1 all products'
// weights are requested at the start.  128-128-128 on 256 rows: 10.4 us,
// forward alone 5.7 (from the FP32 weights 15.9 and 9.7: a layer's 64 KiB came
// no faster than a CU's loads in flight allow, about 1.7 us, however early
// they were issued; the layers as loops of one body 18.9 and 11.6).
template <int D, int T, bool BWD>
__global__ void __launch_bounds__(64 * kRowWaves) mlp_rows_kernel(MlpNet n) {
    constexpr int S = 4 * T, C = 128 * T;
    __shared__ __align__(16) uint16_t act[2][kRows][C + 8];
    __shared__ float zs[kMlpFusedDepth][kRows][C + 1];
    __shared__ float hl[kRows][C + 1];
    __shared__ float gs[kRows];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, r = lane & 15, kg = lane >> 4;
    const int b0 = blockIdx.x * kRows, W = n.W;
    constexpr bool all = T == 1;
    const int64_t layer = mlp_pack_layer(W);
    Weights<S> wf[all ? D : 1], wb[all ? D : 1];  // wb[l]: layer l's, transposed
    if constexpr (all) {
#pragma unroll
        for (int l = 0; l < D; l++) wf[l].load(n.wf + l * layer, w, lane, l == 0 ? n.n_in : W);
        if constexpr (BWD)
#pragma unroll
            for (int l = D - 1; l > 0; l--) wb[l].load(n.wb + l * layer, w, lane, W);
    }
    const float *__restrict__ wh = n.params + n.woff[D];
    float whc[T], whl[2 * T];
#pragma unroll
    for (int t = 0; t < T; t++) whc[t] = wh[min(16 * (w + kRowWaves * t) + r, W - 1)];
#pragma unroll
    for (int i = 0; i < 2 * T; i++) whl[i] = wh[min(lane + 64 * i, W - 1)];
    float bias[D][T];
#pragma unroll
    for (int l = 0; l < D; l++)
#pragma unroll
        for (int t = 0; t < T; t++) bias[l][t] = n.params[n.boff[l] + min(16 * (w + kRowWaves * t) + r, W - 1)];
    const float head_bias = n.params[n.boff[D]];
    float yt[kRows / kRowWaves];
#pragma unroll
    for (int q = 0; q < kRows / kRowWaves; q++) {
        const int b = min(b0 + w + kRowWaves * q, n.B - 1);
        yt[q] = BWD ? n.y[n.rows ? n.rows[b] : b] : 0.0f;
    }
    // the inputs in BF16, zero in the columns past them
    static_assert(64 * kRowWaves == 32 * kRows, "32 threads to a row of inputs");
    {
        const int b = threadIdx.x >> 5;
        const bool live = b0 + b < n.B;
        const int bb = min(b0 + b, n.B - 1);
        const float *__restrict__ xr = n.x + (int64_t)(n.rows ? n.rows[bb] : bb) * n.n_in;
        for (int k = threadIdx.x & 31; k < C; k += 32) {
            uint16_t v = 0;
            if (k < n.n_in) v = live ? bf(xr[k]) : (uint16_t)0;
            act[0][b][k] = v;
            if (BWD && k < n.n_in) n.xt[(int64_t)k * n.bt + b0 + b] = v;
        }
    }
    __syncthreads();
    int cur = 0;
#pragma unroll
    for (int l = 0; l < D; l++) {
        const int K = l == 0 ? n.n_in : W;
#pragma unroll
        for (int t = 0; t < T; t++) {
            const int c = 16 * (w + kRowWaves * t) + r;
            const bool in = c < W;
            Weights<S> &now = wf[all ? l : 0];
            if (!all) now.load(n.wf + l * layer, w + kRowWaves * t, lane, K);
            const floatx4 acc = product(now, &act[cur][r][0], K, kg);
            shortx4 ht;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const float v = acc[e] + bias[l][t], h = silu(v);
                zs[l][4 * kg + e][c] = v;
                const bool live = b0 + 4 * kg + e < n.B;
                ht[e] = live ? bf(h) : (uint16_t)0;
                if (l + 1 < D) {
                    act[cur ^ 1][4 * kg + e][c] = in ? bf(h) : (uint16_t)0;  // zeros past W
                } else {
                    hl[4 * kg + e][c] = h;
                    if (BWD && live && in) n.hlast[(int64_t)(b0 + 4 * kg + e) * W + c] = h;
                }
            }
            if (BWD && l + 1 < D && in)
                *reinterpret_cast<shortx4 *>(n.ht + ((int64_t)l * W + c) * n.bt + b0 + 4 * kg) = ht;
        }
        __syncthreads();
        cur ^= 1;
    }
    // head: a wavefront per row, lane l the columns l, l + 64, ..., a fixed shuffle tree
    {
        float acc[kRows / kRowWaves];
#pragma unroll
        for (int q = 0; q < kRows / kRowWaves; q++) {
            acc[q] = 0.0f;
#pragma unroll
            for (int i = 0; i < 2 * T; i++)
                if (lane + 64 * i < W) acc[q] = fmaf(hl[w + kRowWaves * q][lane + 64 * i], whl[i], acc[q]);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int q = 0; q < kRows / kRowWaves; q++) acc[q] += __shfl_xor(acc[q], o);
        if (lane == 0)
#pragma unroll
            for (int q = 0; q < kRows / kRowWaves; q++) {
                const int b = w + kRowWaves * q;
                const float yh = acc[q] + head_bias;
                float g = 0.0f;
                if (b0 + b < n.B) {
                    n.yhat[b0 + b] = yh;
                    if (BWD) {
                        g = 2.0f * (yh - yt[q]) / (float)n.B;
                        n.g[b0 + b] = g;
                        n.yb[b0 + b] = yt[q];
                    }
                }
                gs[b] = g;
            }
    }
    if constexpr (!BWD) return;
    __syncthreads();
#pragma unroll
    for (int l = D - 1; l >= 0; l--) {
#pragma unroll
        for (int t = 0; t < T; t++) {
            const int c = 16 * (w + kRowWaves * t) + r;
            const bool in = c < W;
            floatx4 d;
            if (l == D - 1) {
#pragma unroll
                for (int e = 0; e < 4; e++) d[e] = gs[4 * kg + e] * whc[t];
            } else {
                Weights<S> &now = wb[all ? l + 1 : 0];
                if (!all) now.load(n.wb + (l + 1) * layer, w + kRowWaves * t, lane, W);
                d = product(now, &act[cur][r][0], W, kg);
            }
            shortx4 dt;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int b = b0 + 4 * kg + e;
                const bool live = b < n.B;
                d[e] = live ? d[e] * dsilu(zs[l][4 * kg + e][c]) : 0.0f;
                dt[e] = bf(d[e]);
                act[cur ^ 1][4 * kg + e][c] = in ? dt[e] : (uint16_t)0;
                if (in && live) n.dz[((int64_t)l * n.B + b) * W + c] = d[e];
            }
            if (in) *reinterpret_cast<shortx4 *>(n.dzt + ((int64_t)l * W + c) * n.bt + b0 + 4 * kg) = dt;
        }
        __syncthreads();
        cur ^= 1;
    }
}

// Gradients, one workgroup (4 wavefronts) each for a 16 x 16 tile of a
// layer's weights, 32 columns of a layer's bias, 32 of the head's weights, or
// the loss, each followed by its parameters' AdamW step.
struct GradBlocks {
    int dw[kMlpFusedDepth + 1];   // first block of layer l's weight tiles; [D]: end
    int bias, head, loss;         // first block of each
};

__global__ void __launch_bounds__(256) mlp_grads_kernel(MlpNet n, GradBlocks G, float *__restrict__ grads,
                                                        float *__restrict__ loss, float *__restrict__ loss_sum,
                                                        MlpAdam A) {
    const int blk = blockIdx.x, W = n.W, D = n.D;
    auto emit = [&](int64_t i, float g) {
        grads[i] = g;
        if (!A.on) return;
        adamw_step(n.params[i], g, A.m[i], A.v[i], A.lr, A.b1, A.b2, A.eps, A.wd, A.c1, A.c2);
    };
    if (blk < G.bias) {
        __shared__ floatx4 part[4][64];
        int l = 0;
        while (blk >= G.dw[l + 1]) l++;
        const int fan = l == 0 ? n.n_in : W, nt = (fan + 15) / 16, t = blk - G.dw[l];
        const int tm = 16 * (t / nt), tn = 16 * (t % nt);
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, r = lane & 15, kg = lane >> 4;
        const uint16_t *__restrict__ a = n.dzt + ((int64_t)l * W + tm + r) * n.bt;
        const uint16_t *__restrict__ b = (l == 0 ? n.xt : n.ht + (int64_t)(l - 1) * W * n.bt) + (int64_t)(tn + r) * n.bt;
        const bool ina = tm + r < W, inb = tn + r < fan;
        auto load = [&](const uint16_t *p, bool in, int k0) {
            const int k = k0 + 8 * kg;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (in && k < n.bt) v = *reinterpret_cast<const uint4 *>(p + k);  // rows past B are stored as zero
            return __builtin_bit_cast(bf16x8, v);
        };
        const int ks = n.B <= 128 ? 1 : 2;
        floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int k0 = 32 * ks * w; k0 < n.B; k0 += 128 * ks) {
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(load(a, ina, k0), load(b, inb, k0), acc, 0, 0, 0);
            if (ks == 2)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(load(a, ina, k0 + 32), load(b, inb, k0 + 32), acc, 0, 0, 0);
        }
        part[w][lane] = acc;
        __syncthreads();
        // thread t: element t / 64 of lane t % 64, so all wavefronts take the optimiser's step
        const float s = ((part[0][lane][w] + part[1][lane][w]) + part[2][lane][w]) + part[3][lane][w];
        const int m = tm + 4 * kg + w, c = tn + r;
        if (m < W && c < fan) {
            const int64_t i = n.woff[l] + (int64_t)m * fan + c;
            emit(i, s);
            if (A.on) pack_weight(n, l, m, c, n.params[i]);
        }
    } else if (blk < G.head) {
        const int per = (W + kSumCols - 1) / kSumCols, l = (blk - G.bias) / per;
        column_sums(n.dz + (int64_t)l * n.B * W, nullptr, n.B, W, false, (blk - G.bias) % per,
                    [&](int i, float s) { emit(n.boff[l] + i, s); });
    } else if (blk < G.loss) {
        column_sums(n.hlast, n.g, n.B, W, true, blk - G.head, [&](int i, float s) { emit(n.woff[D] + i, s); });
    } else {
        __shared__ float part[256];
        float s = 0.0f;
        for (int b = threadIdx.x; b < n.B; b += 256) {
            const float d = n.yhat[b] - n.yb[b];
            s = fmaf(d, d, s);
        }
        part[threadIdx.x] = s;
        __syncthreads();
        for (int h = 128; h > 0; h >>= 1) {
            if ((int)threadIdx.x < h) part[threadIdx.x] += part[threadIdx.x + h];
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            const float v = part[0] / (float)n.B;
            loss[0] = v;
            if (loss_sum) loss_sum[0] += v;
        }
    }
}

template <int D>
void launch_rows_d(const MlpNet &n, bool backward, hipStream_t s) {
    const unsigned blocks = (unsigned)((n.B + kRows - 1) / kRows), threads = 64 * kRowWaves;
    if (n.W > 128)
        backward ? mlp_rows_kernel<D, 2, true><<<blocks, threads, 0, s>>>(n)
                 : mlp_rows_kernel<D, 2, false><<<blocks, threads, 0, s>>>(n);
    else
        backward ? mlp_rows_kernel<D, 1, true><<<blocks, threads, 0, s>>>(n)
                 : mlp_rows_kernel<D, 1, false><<<blocks, threads, 0, s>>>(n);
}

}  // namespace

hipError_t launch_mlp_rows(const MlpNet &n, bool backward, hipStream_t s) {
    if (n.B <= 0) return hipSuccess;
    if (!mlp_fused(1, n.W, n.D) || n.n_in > 64 || n.bt % kRows != 0 || n.bt < n.B || !n.wf) return hipErrorInvalidValue;
    switch (n.D) {
        case 1: launch_rows_d<1>(n, backward, s); break;
        case 2: launch_rows_d<2>(n, backward, s); break;
        case 3: launch_rows_d<3>(n, backward, s); break;
        default: launch_rows_d<4>(n, backward, s); break;
    }
    return hipGetLastError();
}

hipError_t launch_mlp_grads(const MlpNet &n, float *grads, float *loss, float *loss_sum, const MlpAdam &adam,
                            hipStream_t s) {
    if (n.B <= 0) return hipSuccess;
    GradBlocks G{};
    const int mt = (n.W + 15) / 16;
    for (int l = 0; l < n.D; l++) G.dw[l + 1] = G.dw[l] + mt * (((l == 0 ? n.n_in : n.W) + 15) / 16);
    for (int l = n.D; l < kMlpFusedDepth; l++) G.dw[l + 1] = G.dw[l];
    G.bias = G.dw[n.D];
    G.head = G.bias + n.D * ((n.W + kSumCols - 1) / kSumCols);
    G.loss = G.head + (n.W + 1 + kSumCols - 1) / kSumCols;
    mlp_grads_kernel<<<(unsigned)(G.loss + 1), 256, 0, s>>>(n, G, grads, loss, loss_sum, adam);
    return hipGetLastError();
}

}  // namespace gbd
