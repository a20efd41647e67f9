// mlp.hip -- BF16 matrix-core (MFMA) training and inference of the
// warm-start surrogate: a fully connected network with GELU hidden layers,
// mean-squared-error loss and Adam (FP32 master weights), mapping the
// control parameters of a run to its mean wall-normal profiles.
//
// Every product is one "NT" GEMM form, C[m][n] = sum_k A[m][k] * Bt[n][k],
// with A and Bt row-major and K-contiguous, computed by
// v_mfma_f32_16x16x32_bf16 (BF16 inputs, FP32 accumulation):
//   forward   Z  = X  * W       : A = X  [B x in],  Bt = Wt [out x in]
//   input grad dX = dZ * W^T    : A = dZ [B x out], Bt = W  [in x out]
//   weight grad dW = X^T * dZ   : A = Xt [in x B],  Bt = dZt [out x B]
// so weights are kept as BF16 in both [in][out] and [out][in] order and
// activations / gradients in both batch-major and feature-major order.  All
// dimensions are padded to multiples of 32 with zeros that stay zero.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "internal.h"

using namespace nspnp;

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int kMaxLayers = 8;

__device__ __forceinline__ float gelu_f(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float x) {
    return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) + x * 0.39894228040143268f * expf(-0.5f * x * x);
}

enum Epi { EPI_HIDDEN = 0, EPI_OUTPUT = 1, EPI_DX = 2, EPI_DW = 3 };

struct GemmArgs {
    const bf16 *A;   // [M x K]
    const bf16 *Bt;  // [N x K]
    int M, N, K;
    int epi;
    const float *bias;   // HIDDEN, OUTPUT: [N]
    float *Z;            // HIDDEN: pre-activation out [M x N]; DX: pre-activation of the layer below (read)
    bf16 *Y;             // HIDDEN: activation [M x N]; DX: dZ of the layer below [M x N]
    bf16 *Yt;            // HIDDEN / DX: the same, feature-major [N x M]
    float *C;            // OUTPUT: [M x N] FP32 output; DW: [M x N] gradient
};

// One wave per 16 x 16 output tile; 4 waves per block.  kTiled: Bt in tile
// order (tile_at), and the tiles that share columns of it on one XCD, so that
// each XCD's L2 takes its part of the weights.
template <bool kTiled>
__global__ void __launch_bounds__(256) k_gemm_nt(GemmArgs g) {
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int tiles_m = g.M / 16, tiles_n = g.N / 16;
    const int tile = (int)(kTiled ? xcd_tile(blockIdx.x, gridDim.x) : blockIdx.x) * 4 + wave;
    if (tile >= tiles_m * tiles_n) return;
    const int m0 = (kTiled ? tile % tiles_m : tile / tiles_n) * 16, n0 = (kTiled ? tile / tiles_m : tile % tiles_n) * 16;
    const int r = lane & 15, kc = (lane >> 4) * 8;
    const bf16 *pa = g.A + (size_t)(m0 + r) * g.K + kc;
    const bf16 *pb = kTiled ? g.Bt + (size_t)n0 * g.K + lane * 8 : g.Bt + (size_t)(n0 + r) * g.K + kc;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < g.K; k0 += 32) {
        const bf16x8 a = *(const bf16x8 *)(pa + k0);
        const bf16x8 b = *(const bf16x8 *)(pb + (kTiled ? 16 * k0 : k0));
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
    }
    // lane holds rows m0 + 4 (lane / 16) + q, column n0 + lane % 16
    const int n = n0 + r;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int m = m0 + (lane >> 4) * 4 + q;
        const float v = acc[q];
        const size_t o = (size_t)m * g.N + n;
        if (g.epi == EPI_HIDDEN) {
            const float z = v + g.bias[n];
            g.Z[o] = z;
            const bf16 y = (bf16)gelu_f(z);
            g.Y[o] = y;
            g.Yt[(size_t)n * g.M + m] = y;
        } else if (g.epi == EPI_OUTPUT) {
            g.C[o] = v + g.bias[n];
        } else if (g.epi == EPI_DX) {
            const bf16 dz = (bf16)(v * gelu_grad_f(g.Z[o]));
            g.Y[o] = dz;
            g.Yt[(size_t)n * g.M + m] = dz;
        } else {
            g.C[o] = v;
        }
    }
}

// Place of element (n, k) of a B operand [N x K] in the order in which the matrix
// instructions take it: tiles of 16 n and 32 k, in a tile the 8 values of each
// lane.  A wave's load of a tile is then 1 KB in one piece.
__device__ __forceinline__ size_t tile_at(int n, int k, int K) {
    return ((size_t)(n >> 4) * (K >> 5) + (k >> 5)) * 512 + (((k >> 3 & 3) << 4 | (n & 15)) << 3 | (k & 7));
}

// ---- networks whose layers fit one block: two launches a training step ----
// k_net runs the network for 16 rows per block, forward and, for training,
// the loss gradient and the back-propagated dZ of every layer, all of them row-local:
// activations stay in LDS (batch-major, the A operand), 16 waves take the
// 16-column output tiles in turn, and each wave loads the weights of its next
// tile ahead of the barrier between layers.  What the weight gradients need
// (activations and dZ, feature-major) and Z (for GELU') go to memory.
// k_update then forms every layer's weight and bias gradients and, for a
// training step, applies Adam to them in place.  Every sum runs in the order
// of the layer-by-layer kernels (k_gemm_nt, k_bias_grad), so the results are
// the same bit for bit; the loss alone is summed by blocks.
// Bound by latency (layer after layer) and by a block's reads of the weights: in
// tile order a load is one piece of 1 KB; from rows of the matrix it is 16
// pieces of 64 bytes, about 60 cycles each in the one CU that has the block.
// What the last update wrote is in no L2 of another XCD: a training grid of few
// blocks brings kNetAhead more to each XCD that has one of them (blocks go to
// the 8 XCDs in turn), which read the weights once, in the order of their use.
// 64 rows of 3-256-256-256-256-579: a training step 65.7 us with the weights in
// rows, 52.2 in tiles, 47.9 with blocks that read ahead; a forward pass 26.3
// and 16.0.
constexpr int kNetThreads = 1024, kNetWaves = kNetThreads / 64;
constexpr int kNetChunks = 8;  // K chunks of 32 loaded together
constexpr int kNetAhead = 16, kNetAheadBlocks = 64;
constexpr size_t kNetAheadBytes = (size_t)3 << 20;  // of an L2 of 4 MB

struct NetArgs {
    int nl, rows, cols, outs, Bp;  // Bp: row stride of the feature-major arrays
    int ld;                        // row stride of the LDS buffers
    int pd[kMaxLayers + 1];
    const bf16 *wb[kMaxLayers], *wtb[kMaxLayers];     // in tile order (tile_at)
    const float *bias[kMaxLayers];
    float *z[kMaxLayers];                             // feature-major [N x Bp]
    bf16 *actt[kMaxLayers + 1], *dzt[kMaxLayers];
    const float *x, *y;
    float *out;   // forward only: [rows x outs]
    float *part;  // training: sum of squared errors per block
    float scale;  // 2 / (rows outs)
    int blocks;   // of 16 rows; blocks from the next multiple of 8 on read ahead
};

// Reads this wave's share of the weights (1 KB pieces in turn), 8 loads in flight.
__device__ void read_ahead(const NetArgs &a, int first, int stride) {
    const int lane = threadIdx.x & 63, arrays = 2 * a.nl - 1;
    for (int c0 = first; c0 < (int)(kNetAheadBytes >> 10); c0 += 8 * stride) {
        uint4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            int c = c0 + u * stride, q = 0;
            const bf16 *p = a.wtb[0];
            for (; q < arrays; ++q) {
                const int l = q < a.nl ? q : 2 * a.nl - 1 - q;  // wtb forward, then wb backward
                const int n = a.pd[l] * a.pd[l + 1] / 512;      // (widths are multiples of 32)
                p = q < a.nl ? a.wtb[l] : a.wb[l];
                if (c < n) break;
                c -= n;
            }
            v[u] = *((const uint4 *)(q < arrays ? p + (size_t)c * 512 : a.wtb[0]) + lane);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) asm volatile("" ::"v"(v[u].x), "v"(v[u].y), "v"(v[u].z), "v"(v[u].w));
    }
}

template <bool kGrad>
__global__ void __launch_bounds__(kNetThreads) k_net(NetArgs a) {
    extern __shared__ bf16 s_net[];
    __shared__ float s_sum[kNetWaves];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (kGrad && (int)blockIdx.x >= a.blocks) {
        const int q = (int)blockIdx.x - (a.blocks + 7) / 8 * 8;
        if (q >= 0 && q % 8 < a.blocks) read_ahead(a, q / 8 * kNetWaves + wave, kNetAhead * kNetWaves);
        return;
    }
    const int r = lane & 15, kc = (lane >> 4) * 8, mb = (lane >> 4) * 4;
    const int m0 = (int)blockIdx.x * 16, ld = a.ld;
    bf16 *src = s_net, *dst = s_net + 16 * ld;
    // B operand of a tile: rows n0 .. n0 + 15 of W [N x K], chunks k0 .. of 32
    auto load_b = [&](const bf16 *W, int K, int n0, int k0, bf16x8 *b) {
        const bf16 *p = W + (size_t)(n0 * K + k0 * 16) + lane * 8;
#pragma unroll
        for (int q = 0; q < kNetChunks; ++q)
            if (k0 + 32 * q < K) b[q] = *(const bf16x8 *)(p + 512 * q);
    };
    // product of src and one tile, the first chunks of B already in b
    auto tile = [&](const bf16 *W, int K, int n0, bf16x8 *b) -> f32x4 {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int k0 = 0; k0 < K; k0 += 32 * kNetChunks) {
            if (k0) load_b(W, K, n0, k0, b);
            const bf16 *pa = src + r * ld + k0 + kc;
#pragma unroll
            for (int q = 0; q < kNetChunks; ++q)
                if (k0 + 32 * q < K)
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(const bf16x8 *)(pa + 32 * q), b[q], acc, 0, 0, 0);
        }
        return acc;
    };
    bf16x8 b[kNetChunks];
    if (wave < a.pd[1] / 16) load_b(a.wtb[0], a.pd[0], wave * 16, 0, b);
    for (int e = threadIdx.x; e < 16 * a.pd[0]; e += kNetThreads) {
        const int k = e >> 4, m = e & 15;
        const float v = (m0 + m < a.rows && k < a.cols) ? a.x[(size_t)(m0 + m) * a.cols + k] : 0.f;
        const bf16 xb = (bf16)v;
        src[m * ld + k] = xb;
        if (kGrad) a.actt[0][(size_t)k * a.Bp + m0 + m] = xb;
    }
    __syncthreads();
    float sq = 0.f;
    for (int l = 0; l < a.nl; ++l) {
        const int K = a.pd[l], N = a.pd[l + 1];
        const bool last = l == a.nl - 1;
        for (int t = wave; t < N / 16; t += kNetWaves) {
            const int n = t * 16 + r;
            if (t != wave) load_b(a.wtb[l], K, t * 16, 0, b);
            const float bias = a.bias[l][n];
            float yt[4];
            if (kGrad && last) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool in = m0 + mb + q < a.rows && n < a.outs;
                    yt[q] = in ? a.y[(size_t)(m0 + mb + q) * a.outs + n] : 0.f;
                }
            }
            const f32x4 acc = tile(a.wtb[l], K, t * 16, b);
            bf16x4 v;
            f32x4 zv;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int m = mb + q;
                const float z = acc[q] + bias;
                zv[q] = z;
                if (!last) {
                    v[q] = (bf16)gelu_f(z);
                } else if (kGrad) {
                    float g = 0.f;
                    if (m0 + m < a.rows && n < a.outs) {
                        const float d = z - yt[q];
                        sq += d * d;
                        g = a.scale * d;
                    }
                    v[q] = (bf16)g;
                } else if (m0 + m < a.rows && n < a.outs) {
                    a.out[(size_t)(m0 + m) * a.outs + n] = z;
                }
                if (kGrad || !last) dst[m * ld + n] = v[q];
            }
            if (kGrad) {
                const size_t o = (size_t)n * a.Bp + m0 + mb;
                if (!last) *(f32x4 *)(a.z[l] + o) = zv;
                *(bf16x4 *)((last ? a.dzt[l] : a.actt[l + 1]) + o) = v;
            }
        }
        // the next layer's (or the backward pass's first) weights
        if (!last) {
            if (wave < a.pd[l + 2] / 16) load_b(a.wtb[l + 1], N, wave * 16, 0, b);
        } else if (kGrad && l > 0) {
            if (wave < K / 16) load_b(a.wb[l], N, wave * 16, 0, b);
        }
        __syncthreads();
        bf16 *sw = src;
        src = dst;
        dst = sw;
    }
    if (!kGrad) return;
    for (int l = a.nl - 1; l > 0; --l) {
        const int K = a.pd[l + 1], N = a.pd[l];
        for (int t = wave; t < N / 16; t += kNetWaves) {
            const int n = t * 16 + r;
            const size_t o = (size_t)n * a.Bp + m0 + mb;
            const f32x4 zv = *(const f32x4 *)(a.z[l - 1] + o);  // (this thread's own stores)
            if (t != wave) load_b(a.wb[l], K, t * 16, 0, b);
            const f32x4 acc = tile(a.wb[l], K, t * 16, b);
            bf16x4 v;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[q] = (bf16)(acc[q] * gelu_grad_f(zv[q]));
                dst[(mb + q) * ld + n] = v[q];
            }
            *(bf16x4 *)(a.dzt[l - 1] + o) = v;
        }
        if (l > 1 && wave < a.pd[l - 1] / 16) load_b(a.wb[l - 1], N, wave * 16, 0, b);
        __syncthreads();
        bf16 *sw = src;
        src = dst;
        dst = sw;
    }
    for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
    if (lane == 0) s_sum[wave] = sq;
    __syncthreads();
    if (threadIdx.x == 0) {
        float s = 0.f;
        for (int w = 0; w < kNetWaves; ++w) s += s_sum[w];
        a.part[blockIdx.x] = s;
    }
}

// Adam on one FP32 master weight (the multiply-add order is written out, so
// that every kernel using it rounds alike).
struct AdamStep {
    float lr, b1, b2, eps, c1, c2;
};
__device__ __forceinline__ float adam_element(const AdamStep &s, float w, float &m, float &v, float g) {
    m = __builtin_fmaf(1.f - s.b1, g, s.b1 * m);
    v = __builtin_fmaf(g, (1.f - s.b2) * g, s.b2 * v);
    return w - s.lr * (m / s.c1) / (sqrtf(v / s.c2) + s.eps);
}

struct UpdateArgs {
    int nl, Bp, K;  // K: batch rows summed (multiple of 32), Bp their stride
    int pd[kMaxLayers + 1];
    int first[kMaxLayers + 1];  // first wave of each layer: its weight tiles, then its bias columns by 64
    const bf16 *actt[kMaxLayers], *dzt[kMaxLayers];
    float *w[kMaxLayers], *m[kMaxLayers], *v[kMaxLayers], *g[kMaxLayers];
    bf16 *wb[kMaxLayers], *wtb[kMaxLayers];
    int apply;  // 0: gradients only
    AdamStep s;
    const float *part;
    int nparts;
    float count;  // rows * outs
    float *loss, *loss2;  // loss2: the caller's (may be NULL)
};

__global__ void __launch_bounds__(256) k_update(UpdateArgs a) {
    const int lane = threadIdx.x & 63;
    const int job = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (job > a.first[a.nl]) return;
    if (job == a.first[a.nl]) {  // the loss, block sums in order
        float s = 0.f;
        for (int p = lane; p < a.nparts; p += 64) s += a.part[p];
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if (lane == 0) {
            s /= a.count;
            *a.loss = s;
            if (a.loss2) *a.loss2 = s;
        }
        return;
    }
    int l = 0;
    while (job >= a.first[l + 1]) ++l;
    const int M = a.pd[l], N = a.pd[l + 1], tn = N / 16, t = job - a.first[l];
    float *w = a.w[l], *mo = a.m[l], *ve = a.v[l], *g = a.g[l];
    if (t >= (M / 16) * tn) {  // bias columns
        const int n = (t - (M / 16) * tn) * 64 + lane;
        if (n >= N) return;
        const bf16 *p = a.dzt[l] + (size_t)n * a.Bp;
        float s = 0.f;
        for (int k = 0; k < a.K; k += 32) {
            bf16x8 v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = *(const bf16x8 *)(p + k + 8 * q);
#pragma unroll
            for (int q = 0; q < 32; ++q) s += (float)v[q >> 3][q & 7];
        }
        const size_t o = (size_t)M * N + n;
        g[o] = s;
        if (a.apply) w[o] = adam_element(a.s, w[o], mo[o], ve[o], s);
        return;
    }
    const int m0 = (t / tn) * 16, n0 = (t % tn) * 16;
    const int r = lane & 15, kc = (lane >> 4) * 8, m = m0 + (lane >> 4) * 4, n = n0 + r;
    float ww[4], wm[4], wv[4];
    if (a.apply) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const size_t o = (size_t)(m + q) * N + n;
            ww[q] = w[o];
            wm[q] = mo[o];
            wv[q] = ve[o];
        }
    }
    const bf16 *pa = a.actt[l] + (size_t)(m0 + r) * a.Bp + kc, *pb = a.dzt[l] + (size_t)(n0 + r) * a.Bp + kc;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < a.K; k0 += 32)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(const bf16x8 *)(pa + k0), *(const bf16x8 *)(pb + k0), acc, 0, 0, 0);
    bf16x4 wt;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const size_t o = (size_t)(m + q) * N + n;
        g[o] = acc[q];
        if (a.apply) {
            const float wn = adam_element(a.s, ww[q], wm[q], wv[q], acc[q]);
            w[o] = wn;
            mo[o] = wm[q];
            ve[o] = wv[q];
            wt[q] = (bf16)wn;
            a.wb[l][tile_at(m + q, n, N)] = wt[q];
        }
    }
    if (a.apply) *(bf16x4 *)(a.wtb[l] + tile_at(n, m, M)) = wt;
}

// Loss and output-layer gradient: mean over the valid rows and outputs of
// (yhat - y)^2; dZ = 2 (yhat - y) / (rows * outs), zero in the padding.
__global__ void __launch_bounds__(256) k_loss(const float *yhat, const float *y, int rows, int outs, int Bp, int Np,
                                              bf16 *dz, bf16 *dzt, float *loss) {
    __shared__ float s[256];
    float acc = 0.f;
    const float scale = 2.0f / ((float)rows * (float)outs);
    for (int e = threadIdx.x; e < Bp * Np; e += blockDim.x) {
        const int m = e / Np, n = e - m * Np;
        float g = 0.f;
        if (m < rows && n < outs) {
            const float d = yhat[e] - y[(size_t)m * outs + n];
            acc += d * d;
            g = scale * d;
        }
        const bf16 gb = (bf16)g;
        dz[e] = gb;
        dzt[(size_t)n * Bp + m] = gb;
    }
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = s[0] / ((float)rows * (float)outs);
}

// bias gradient: column sums of dZ over the batch
__global__ void k_bias_grad(const bf16 *dzt, int Bp, int Np, float *db) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= Np) return;
    float s = 0.f;
    for (int m = 0; m < Bp; ++m) s += (float)dzt[(size_t)n * Bp + m];
    db[n] = s;
}

// Adam on FP32 master weights, then BF16 copies in both orders.
struct AdamArgs {
    float *w, *m, *v;   // master / moments, [in_p x out_p] followed by [out_p] bias
    const float *g;     // gradients in the same layout
    bf16 *wb, *wtb;     // BF16 weights [in_p][out_p] and [out_p][in_p]
    int in_p, out_p;
    AdamStep s;
};

__global__ void __launch_bounds__(256) k_adam(AdamArgs a) {
    const int nW = a.in_p * a.out_p;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nW + a.out_p) return;
    const float w = adam_element(a.s, a.w[e], a.m[e], a.v[e], a.g[e]);
    a.w[e] = w;
    if (e < nW) {
        const int i = e / a.out_p, o = e - i * a.out_p;
        const bf16 wb = (bf16)w;
        a.wb[e] = wb;
        a.wtb[(size_t)o * a.in_p + i] = wb;
    }
}

// FP32 rows [rows x cols] -> padded BF16 [Bp x Kp] and [Kp x Bp]
__global__ void k_pack_input(const float *x, int rows, int cols, int Bp, int Kp, bf16 *xb, bf16 *xtb) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= Bp * Kp) return;
    const int m = e / Kp, k = e - m * Kp;
    const float v = (m < rows && k < cols) ? x[(size_t)m * cols + k] : 0.f;
    const bf16 b = (bf16)v;
    xb[e] = b;
    xtb[(size_t)k * Bp + m] = b;
}

// copy the valid part of the FP32 output [Bp x Np] to [rows x outs]
__global__ void k_unpack_output(const float *yp, int rows, int outs, int Np, float *y) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= rows * outs) return;
    const int m = e / outs, n = e - m * outs;
    y[e] = yp[(size_t)m * Np + n];
}

// tiled: the copies in tile order, for k_net; else [in_p][out_p] and [out_p][in_p]
__global__ void k_sync_bf16(const float *w, int in_p, int out_p, bf16 *wb, bf16 *wtb, int tiled) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= in_p * out_p) return;
    const int i = e / out_p, o = e - i * out_p;
    const bf16 b = (bf16)w[e];
    wb[tiled ? tile_at(i, o, out_p) : (size_t)e] = b;
    wtb[tiled ? tile_at(o, i, in_p) : (size_t)o * in_p + i] = b;
}

int pad32(int n) { return (n + 31) / 32 * 32; }

}  // namespace

struct nspnp_mlp {
    int nl;                      // number of weight layers
    int sizes[kMaxLayers + 1];   // unpadded widths
    int padded[kMaxLayers + 1];  // padded to 32
    int Bp, Bmax;                // padded batch rows
    bool fused;                  // k_net / k_update (net_fits), else layer by layer
    int ld;                      // row stride of k_net's LDS buffers
    hipStream_t stream;
    float *w[kMaxLayers], *m[kMaxLayers], *v[kMaxLayers], *g[kMaxLayers];  // each [in_p*out_p + out_p]
    bf16 *wb[kMaxLayers], *wtb[kMaxLayers];
    bf16 *act[kMaxLayers + 1], *actt[kMaxLayers + 1];  // act[0] = input
    float *z[kMaxLayers];
    float *yhat;
    bf16 *dz[kMaxLayers], *dzt[kMaxLayers];
    float *loss;
    int64_t t;
};

namespace {

// Two row-major LDS buffers of 16 rows (8 values of padding a row spread the
// banks), for layers of up to 768: training steps through 8 layers of 768 take
// 0.85 (1 row), 0.64 (64) and 0.13 (1024) of their time layer by layer.  Wider
// networks run layer by layer: forward passes through 5 layers of 992 (which
// fit 64 KB too) 95 and 58 us.
size_t net_lds(int widest) { return 2 * 16 * (size_t)(widest + 8) * sizeof(bf16); }
bool net_fits(int widest) { return widest <= 768; }

size_t mlp_layout(int nl, const int *sizes, int batch, nspnp_mlp *h, char *base) {
    size_t o = 0;
    auto take = [&](size_t bytes) {
        char *p = base ? base + o : nullptr;
        o = (o + bytes + 255) & ~(size_t)255;
        return p;
    };
    int pd[kMaxLayers + 1];
    for (int l = 0; l <= nl; ++l) pd[l] = pad32(sizes[l]);
    const int Bp = pad32(batch);
    for (int l = 0; l < nl; ++l) {
        const size_t np = (size_t)pd[l] * pd[l + 1] + pd[l + 1];
        float *w = (float *)take(np * 4), *m = (float *)take(np * 4), *v = (float *)take(np * 4);
        float *g = (float *)take(np * 4);
        bf16 *wb = (bf16 *)take((size_t)pd[l] * pd[l + 1] * 2), *wtb = (bf16 *)take((size_t)pd[l] * pd[l + 1] * 2);
        if (h) {
            h->w[l] = w; h->m[l] = m; h->v[l] = v; h->g[l] = g; h->wb[l] = wb; h->wtb[l] = wtb;
        }
    }
    for (int l = 0; l <= nl; ++l) {
        bf16 *a = (bf16 *)take((size_t)Bp * pd[l] * 2), *at = (bf16 *)take((size_t)Bp * pd[l] * 2);
        if (h) { h->act[l] = a; h->actt[l] = at; }
    }
    for (int l = 0; l < nl; ++l) {
        float *zz = (float *)take((size_t)Bp * pd[l + 1] * 4);
        bf16 *d = (bf16 *)take((size_t)Bp * pd[l + 1] * 2), *dt = (bf16 *)take((size_t)Bp * pd[l + 1] * 2);
        if (h) { h->z[l] = zz; h->dz[l] = d; h->dzt[l] = dt; }
    }
    float *yh = (float *)take((size_t)Bp * pd[nl] * 4);
    float *ls = (float *)take(4 * (size_t)(64 + Bp / 16));  // the loss, then k_net's block sums
    if (h) {
        h->yhat = yh;
        h->loss = ls;
        h->nl = nl;
        h->Bp = Bp;
        h->Bmax = batch;
        for (int l = 0; l <= nl; ++l) { h->sizes[l] = sizes[l]; h->padded[l] = pd[l]; }
        int widest = 0;
        for (int l = 0; l <= nl; ++l) widest = std::max(widest, pd[l]);
        h->ld = widest + 8;
        h->fused = net_fits(widest);
    }
    return o;
}

int check_mlp(int nl, const int *sizes, int batch) {
    if (nl < 1 || nl > kMaxLayers || !sizes || batch < 1 || batch > 4096)
        return fail_code(NSPNP_ERR_INVALID, "mlp: 1..8 layers and 1..4096 rows");
    for (int l = 0; l <= nl; ++l)
        if (sizes[l] < 1 || sizes[l] > 8192) return fail_code(NSPNP_ERR_INVALID, "mlp: widths must be 1..8192");
    return NSPNP_OK;
}

#define M_TRY(expr)                                                                                       \
    do {                                                                                                  \
        hipError_t e_ = (expr);                                                                           \
        if (e_ != hipSuccess) return fail_code(NSPNP_ERR_HIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

hipError_t gemm(nspnp_mlp *h, const GemmArgs &g, bool tiled = false) {
    const int tiles = (g.M / 16) * (g.N / 16);
    if (tiled) k_gemm_nt<true><<<(tiles + 3) / 4, 256, 0, h->stream>>>(g);
    else k_gemm_nt<false><<<(tiles + 3) / 4, 256, 0, h->stream>>>(g);
    return hipGetLastError();
}

// Bp: batch rows packed and run, a multiple of 32
int pack_input(nspnp_mlp *h, const float *x, int rows, int Bp) {
    const int n = Bp * h->padded[0];
    k_pack_input<<<(n + 255) / 256, 256, 0, h->stream>>>(x, rows, h->sizes[0], Bp, h->padded[0], h->act[0],
                                                         h->actt[0]);
    M_TRY(hipGetLastError());
    return NSPNP_OK;
}

int forward(nspnp_mlp *h, int Bp) {
    for (int l = 0; l < h->nl; ++l) {
        GemmArgs g{};
        g.A = h->act[l];
        g.Bt = h->wtb[l];
        g.M = Bp;
        g.N = h->padded[l + 1];
        g.K = h->padded[l];
        g.bias = h->w[l] + (size_t)h->padded[l] * h->padded[l + 1];
        if (l < h->nl - 1) {
            g.epi = EPI_HIDDEN;
            g.Z = h->z[l];
            g.Y = h->act[l + 1];
            g.Yt = h->actt[l + 1];
        } else {
            g.epi = EPI_OUTPUT;
            g.C = h->yhat;
        }
        M_TRY(gemm(h, g, h->fused));
    }
    return NSPNP_OK;
}

// gradients of the loss for the rows currently packed (requires forward)
int backward(nspnp_mlp *h, const float *y, int rows) {
    const int L = h->nl;
    k_loss<<<1, 256, 0, h->stream>>>(h->yhat, y, rows, h->sizes[L], h->Bp, h->padded[L], h->dz[L - 1],
                                     h->dzt[L - 1], h->loss);
    M_TRY(hipGetLastError());
    for (int l = L - 1; l >= 0; --l) {
        const int in_p = h->padded[l], out_p = h->padded[l + 1];
        GemmArgs gw{};
        gw.A = h->actt[l];
        gw.Bt = h->dzt[l];
        gw.M = in_p;
        gw.N = out_p;
        gw.K = h->Bp;
        gw.epi = EPI_DW;
        gw.C = h->g[l];
        M_TRY(gemm(h, gw));
        k_bias_grad<<<(out_p + 255) / 256, 256, 0, h->stream>>>(h->dzt[l], h->Bp, out_p,
                                                                h->g[l] + (size_t)in_p * out_p);
        M_TRY(hipGetLastError());
        if (l > 0) {
            GemmArgs gx{};
            gx.A = h->dz[l];
            gx.Bt = h->wb[l];
            gx.M = h->Bp;
            gx.N = in_p;
            gx.K = out_p;
            gx.epi = EPI_DX;
            gx.Z = h->z[l - 1];
            gx.Y = h->dz[l - 1];
            gx.Yt = h->dzt[l - 1];
            M_TRY(gemm(h, gx));
        }
    }
    return NSPNP_OK;
}

// Forward passes of up to 384 rows go layer by layer, from the weights in tile
// order, where k_net's 16 waves wait longer for weights than its launches
// save: a wave loads a layer's weights in ceil(N / 256) tiles of ceil(K / 256)
// pieces, one after the other, and nearly all layers have 3 x 3 of them; or the
// weights (BF16) don't fit an XCD's 4 MB of L2, each of which reads them all.
// 64 rows: 1 layer of 768 12 us (k_net 18), 3 of 704 29 (34), 5 of 640 44 (62),
// 8 of 768 75 (126), 8 of 512 58 (59); k_net stays ahead on 3 layers of 512 (21
// against 24), 8-768-768-8 (17, 23) and 5 layers of 8-640-..-8 (29, 38).  More
// rows give k_net more blocks: 4 layers of 576, 256 rows 36 (35), 384 rows 37
// (35), 512 rows 43 (35); 8 of 640, 384 rows 78 (98), 512 rows 85 (97).
constexpr int kLayerRows = 384;
bool forward_by_layers(const nspnp_mlp *h, int rows) {
    int64_t weights = 0;
    int pieces = 0;
    for (int l = 0; l < h->nl; ++l) {
        weights += (int64_t)h->padded[l] * h->padded[l + 1];
        pieces += ((h->padded[l] + 255) / 256) * ((h->padded[l + 1] + 255) / 256);
    }
    return rows <= kLayerRows && (2 * weights > 3800000 || pieces > 7 * h->nl);
}

// k_net on the handle's weights: forward into out, or (out NULL) forward and
// backward towards y.
int run_net(nspnp_mlp *h, const float *x, const float *y, int rows, float *out) {
    NetArgs a{};
    a.nl = h->nl;
    a.rows = rows;
    a.cols = h->sizes[0];
    a.outs = h->sizes[h->nl];
    a.Bp = h->Bp;
    a.ld = h->ld;
    for (int l = 0; l <= h->nl; ++l) {
        a.pd[l] = h->padded[l];
        a.actt[l] = h->actt[l];
    }
    for (int l = 0; l < h->nl; ++l) {
        a.wb[l] = h->wb[l];
        a.wtb[l] = h->wtb[l];
        a.bias[l] = h->w[l] + (size_t)h->padded[l] * h->padded[l + 1];
        a.z[l] = h->z[l];
        a.dzt[l] = h->dzt[l];
    }
    a.x = x;
    a.y = y;
    a.out = out;
    a.part = h->loss + 64;
    a.scale = 2.0f / ((float)rows * (float)a.outs);
    const size_t lds = net_lds(h->ld - 8);
    a.blocks = pad32(rows) / 16;
    // (more blocks share what they read; a forward pass finds the weights of
    // the one before it: 16 us with 64 rows, 19 with blocks that read ahead)
    const int grid = a.blocks <= kNetAheadBlocks ? (a.blocks + 7) / 8 * 8 + 8 * kNetAhead : a.blocks;
    if (out) k_net<false><<<(rows + 15) / 16, kNetThreads, lds, h->stream>>>(a);
    else k_net<true><<<grid, kNetThreads, lds, h->stream>>>(a);
    M_TRY(hipGetLastError());
    return NSPNP_OK;
}

// Weight and bias gradients of the rows that k_net ran, and (apply) Adam.
int run_update(nspnp_mlp *h, int rows, const AdamStep *s, float *dev_loss) {
    UpdateArgs a{};
    a.nl = h->nl;
    a.Bp = h->Bp;
    a.K = pad32(rows);
    int jobs = 0;
    for (int l = 0; l < h->nl; ++l) {
        a.first[l] = jobs;
        jobs += (h->padded[l] / 16) * (h->padded[l + 1] / 16) + (h->padded[l + 1] + 63) / 64;
        a.actt[l] = h->actt[l];
        a.dzt[l] = h->dzt[l];
        a.w[l] = h->w[l]; a.m[l] = h->m[l]; a.v[l] = h->v[l]; a.g[l] = h->g[l];
        a.wb[l] = h->wb[l]; a.wtb[l] = h->wtb[l];
    }
    a.first[h->nl] = jobs;  // one more wave: the loss
    for (int l = 0; l <= h->nl; ++l) a.pd[l] = h->padded[l];
    a.apply = s != nullptr;
    if (s) a.s = *s;
    a.part = h->loss + 64;
    a.nparts = a.K / 16;
    a.count = (float)rows * (float)h->sizes[h->nl];
    a.loss = h->loss;
    a.loss2 = dev_loss;
    k_update<<<(jobs + 1 + 3) / 4, 256, 0, h->stream>>>(a);
    M_TRY(hipGetLastError());
    return NSPNP_OK;
}

}  // namespace

extern "C" {

size_t nspnp_mlp_workspace_bytes(int32_t n_layers, const int32_t *sizes, int32_t max_rows) {
    if (check_mlp(n_layers, sizes, max_rows)) return 0;
    return mlp_layout(n_layers, sizes, max_rows, nullptr, nullptr);
}

int nspnp_mlp_init(int32_t n_layers, const int32_t *sizes, int32_t max_rows, const float *host_params,
                   void *dev_workspace, size_t bytes, void *hip_stream, nspnp_mlp **out) {
    if (!out || !host_params) return fail_code(NSPNP_ERR_INVALID, "mlp_init: NULL argument");
    *out = nullptr;
    int rc = check_mlp(n_layers, sizes, max_rows);
    if (rc) return rc;
    const size_t need = mlp_layout(n_layers, sizes, max_rows, nullptr, nullptr);
    if (!dev_workspace || bytes < need || ((uintptr_t)dev_workspace & 255))
        return fail_code(NSPNP_ERR_WORKSPACE, "mlp workspace missing, too small or misaligned");
    nspnp_mlp *h = new nspnp_mlp();
    mlp_layout(n_layers, sizes, max_rows, h, (char *)dev_workspace);
    h->stream = (hipStream_t)hip_stream;
    h->t = 0;
    // zero everything (padding must stay zero), then the parameters
    std::vector<char> zeros(need, 0);
    hipError_t e = hipMemcpyAsync(dev_workspace, zeros.data(), need, hipMemcpyHostToDevice, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) {
        delete h;
        return fail_code(NSPNP_ERR_HIP, std::string("mlp init: ") + hipGetErrorString(e));
    }
    *out = h;
    return nspnp_mlp_set_params(h, host_params);
}

// parameters as W_0 [in x out] row-major, b_0 [out], W_1, b_1, ... (FP32)
int nspnp_mlp_set_params(nspnp_mlp *h, const float *host_params) {
    if (!h || !host_params) return fail_code(NSPNP_ERR_INVALID, "mlp_set_params: NULL argument");
    const float *src = host_params;
    for (int l = 0; l < h->nl; ++l) {
        const int in = h->sizes[l], out = h->sizes[l + 1], in_p = h->padded[l], out_p = h->padded[l + 1];
        std::vector<float> buf((size_t)in_p * out_p + out_p, 0.f);
        for (int i = 0; i < in; ++i)
            for (int o = 0; o < out; ++o) buf[(size_t)i * out_p + o] = src[(size_t)i * out + o];
        src += (size_t)in * out;
        for (int o = 0; o < out; ++o) buf[(size_t)in_p * out_p + o] = src[o];
        src += out;
        M_TRY(hipMemcpyAsync(h->w[l], buf.data(), buf.size() * 4, hipMemcpyHostToDevice, h->stream));
        M_TRY(hipStreamSynchronize(h->stream));
        k_sync_bf16<<<(in_p * out_p + 255) / 256, 256, 0, h->stream>>>(h->w[l], in_p, out_p, h->wb[l], h->wtb[l],
                                                                           h->fused ? 1 : 0);
        M_TRY(hipGetLastError());
    }
    M_TRY(hipStreamSynchronize(h->stream));
    return NSPNP_OK;
}

int nspnp_mlp_get_params(nspnp_mlp *h, float *host_params, float *host_grads) {
    if (!h || (!host_params && !host_grads)) return fail_code(NSPNP_ERR_INVALID, "mlp_get_params: NULL argument");
    size_t off = 0;
    for (int l = 0; l < h->nl; ++l) {
        const int in = h->sizes[l], out = h->sizes[l + 1], in_p = h->padded[l], out_p = h->padded[l + 1];
        std::vector<float> buf((size_t)in_p * out_p + out_p);
        for (int which = 0; which < 2; ++which) {
            float *dst = which == 0 ? host_params : host_grads;
            if (!dst) continue;
            M_TRY(hipMemcpyAsync(buf.data(), which == 0 ? h->w[l] : h->g[l], buf.size() * 4, hipMemcpyDeviceToHost,
                                 h->stream));
            M_TRY(hipStreamSynchronize(h->stream));
            for (int i = 0; i < in; ++i)
                for (int o = 0; o < out; ++o) dst[off + (size_t)i * out + o] = buf[(size_t)i * out_p + o];
            for (int o = 0; o < out; ++o) dst[off + (size_t)in * out + o] = buf[(size_t)in_p * out_p + o];
        }
        off += (size_t)in * out + out;
    }
    return NSPNP_OK;
}

int nspnp_mlp_forward(nspnp_mlp *h, const float *dev_x, int32_t rows, float *dev_y) {
    if (!h || !dev_x || !dev_y || rows < 1 || rows > h->Bmax) return fail_code(NSPNP_ERR_INVALID, "mlp_forward: bad rows");
    if (h->fused && !forward_by_layers(h, rows)) {
        // blocks write their rows of dev_y while others still read theirs of
        // dev_x: an output that overlaps the input goes through the workspace
        const uintptr_t x0 = (uintptr_t)dev_x, y0 = (uintptr_t)dev_y;
        const size_t nx = (size_t)rows * h->sizes[0] * 4, ny = (size_t)rows * h->sizes[h->nl] * 4;
        const bool over = x0 < y0 + ny && y0 < x0 + nx;
        const int rn = run_net(h, dev_x, nullptr, rows, over ? h->yhat : dev_y);
        if (rn || !over) return rn;
        M_TRY(hipMemcpyAsync(dev_y, h->yhat, ny, hipMemcpyDeviceToDevice, h->stream));
        return NSPNP_OK;
    }
    const int Bp = h->fused ? pad32(rows) : h->Bp;
    int rc = pack_input(h, dev_x, rows, Bp);
    if (rc || (rc = forward(h, Bp))) return rc;
    const int n = rows * h->sizes[h->nl];
    k_unpack_output<<<(n + 255) / 256, 256, 0, h->stream>>>(h->yhat, rows, h->sizes[h->nl], h->padded[h->nl], dev_y);
    M_TRY(hipGetLastError());
    return NSPNP_OK;
}

int nspnp_mlp_gradients(nspnp_mlp *h, const float *dev_x, const float *dev_y, int32_t rows, float *loss) {
    if (!h || !dev_x || !dev_y || rows < 1 || rows > h->Bmax) return fail_code(NSPNP_ERR_INVALID, "mlp_gradients: bad rows");
    int rc;
    if (h->fused) rc = run_net(h, dev_x, dev_y, rows, nullptr), rc = rc ? rc : run_update(h, rows, nullptr, nullptr);
    else rc = pack_input(h, dev_x, rows, h->Bp), rc = rc ? rc : forward(h, h->Bp), rc = rc ? rc : backward(h, dev_y, rows);
    if (rc) return rc;
    if (loss) {
        M_TRY(hipMemcpyAsync(loss, h->loss, 4, hipMemcpyDeviceToHost, h->stream));
        M_TRY(hipStreamSynchronize(h->stream));
    }
    return NSPNP_OK;
}

int nspnp_mlp_train_step(nspnp_mlp *h, const float *dev_x, const float *dev_y, int32_t rows, float lr,
                         float *dev_loss) {
    if (!h || !dev_x || !dev_y || rows < 1 || rows > h->Bmax) return fail_code(NSPNP_ERR_INVALID, "mlp_train_step: bad rows");
    const double t = (double)(h->t + 1);
    const AdamStep step{lr, 0.9f, 0.999f, 1e-8f, (float)(1.0 - std::pow(0.9, t)), (float)(1.0 - std::pow(0.999, t))};
    int rc;
    if (h->fused) {
        if ((rc = run_net(h, dev_x, dev_y, rows, nullptr))) return rc;
        h->t += 1;
        return run_update(h, rows, &step, dev_loss);
    }
    if ((rc = pack_input(h, dev_x, rows, h->Bp)) || (rc = forward(h, h->Bp)) || (rc = backward(h, dev_y, rows))) return rc;
    h->t += 1;
    AdamArgs a{};
    a.s = step;
    for (int l = 0; l < h->nl; ++l) {
        a.w = h->w[l]; a.m = h->m[l]; a.v = h->v[l]; a.g = h->g[l];
        a.wb = h->wb[l]; a.wtb = h->wtb[l];
        a.in_p = h->padded[l];
        a.out_p = h->padded[l + 1];
        const int n = a.in_p * a.out_p + a.out_p;
        k_adam<<<(n + 255) / 256, 256, 0, h->stream>>>(a);
        M_TRY(hipGetLastError());
    }
    if (dev_loss) M_TRY(hipMemcpyAsync(dev_loss, h->loss, 4, hipMemcpyDeviceToDevice, h->stream));
    return NSPNP_OK;
}

int nspnp_mlp_sync(nspnp_mlp *h) {
    if (!h) return fail_code(NSPNP_ERR_INVALID, "mlp is NULL");
    M_TRY(hipStreamSynchronize(h->stream));
    return NSPNP_OK;
}

void nspnp_mlp_destroy(nspnp_mlp *h) { delete h; }

}  // extern "C"
