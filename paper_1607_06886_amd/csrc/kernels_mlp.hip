// Learned sampling proposal: BF16 MLP forward/backward on MFMA (FP32
// accumulation), mixture negative log-likelihood, Adam, mixture sampling.
#include <hip/hip_runtime.h>
#include <math.h>

#include "mlp_internal.hpp"

namespace pump {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // (a caller's rows)

__device__ __forceinline__ uint16_t f2bf(float f) {
    // round to nearest even; NaN stays NaN
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// ---------------------------------------------------------------------------
// The network over its batch rows.  A workgroup of 8 waves takes 16 RT rows
// through every layer (and, in training, back), their activations in LDS and
// the weights from L2: a layer is 16 RT x 256 outputs over K = 256 or 416, so
// the products of a 2048-row batch are some 4 us of matrix work, and what
// counts is the chain of layers: launches between them, and a workgroup's
// weights arriving (a layer's 128 KB at what one CU reads from L2), which are
// asked for a layer ahead.  The layers are a loop where they can be.  Before,
// each layer was a launch of 64 x 64 tiles with its activations written twice
// to memory (row- and column-major), and the bias gradients one thread's walk
// over the batch: a 4999-row forward took 100 us (now 31, 19 of them on the
// device), a 2048-row training step 2.5 ms (now 67 us: rows 27, weight
// gradients 10, Adam 5.5).
//
// Products are v_mfma_f32_16x16x32_bf16 over k = 0, 32, ... in order.  Lane l
// feeds row l % 16 and k = 8 (l / 16) .. +7 of each operand; it receives
// D[4 (l / 16) + r][l % 16], r = 0..3.
// ---------------------------------------------------------------------------
constexpr int kRowThreads = 512;
constexpr int kLdIn = kInPad + 8;     // LDS rows padded by 16 bytes against bank conflicts
constexpr int kLdHid = kHidden + 8;
constexpr int kLdOut = kOutPad + 4;   // FP32 outputs / output gradients

// Operands lie in memory as the lanes read them ("fragment order"): the 16 x 32
// tile of rows n / 16 and k / 32 is 1 KB, lane after lane, so that a wave's load
// is contiguous.  With plain rows a lane's neighbours lay a row apart, and a
// 2048-row forward took 29.7 us instead of 13.5, its training step 48 + 25.6
// (rows, weight gradients) instead of 27 + 10.
__device__ __forceinline__ size_t frag_at(int n, int k, int nk) {
    return ((((size_t)(n >> 4) * nk + (k >> 5)) * 64 + (n & 15) + 16 * ((k >> 3) & 3)) << 3) + (k & 7);
}

// A wave's share of a layer's weights: column tiles 2 * wave and 2 * wave + 1
// over K = 32 NK.
template <int NK>
struct Frags {
    bf16x8 b[2][NK];
};

// All of it in flight at once; it does not depend on the activations, so it is
// asked for a layer ahead.
template <int NK>
__device__ __forceinline__ void load_frags(const uint16_t* __restrict__ Bm, int n_tiles, Frags<NK>& f) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int tile = min(2 * wave + j, n_tiles - 1);
        const bf16x8* q = reinterpret_cast<const bf16x8*>(Bm) + (size_t)tile * NK * 64 + lane;
#pragma unroll
        for (int k = 0; k < NK; ++k) f.b[j][k] = q[64 * k];
    }
    __builtin_amdgcn_sched_barrier(0);
}

// acc[j][i]: column tile 2 * wave + j, row tile i of s_a (LDS, 32 NK wide).
template <int RT, int NK>
__device__ __forceinline__ void rows_product(const uint16_t* s_a, int lda, const Frags<NK>& f,
                                             f32x4 (&acc)[2][RT]) {
    const int lane = threadIdx.x & 63;
    const int r = lane & 15, kq = (lane >> 4) * 8;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < RT; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < NK; ++k)
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            const bf16x8 a = *reinterpret_cast<const bf16x8*>(s_a + (16 * i + r) * lda + 32 * k + kq);
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, f.b[j][k], acc[j][i], 0, 0, 0);
        }
}

// Condition rows m0 .. m0 + R - 1 as BF16 in LDS, zero past the batch and the
// condition's width.
template <int R>
__device__ __forceinline__ void load_rows(const float* __restrict__ X, int B, int m0, uint16_t* s_in) {
    constexpr int kGroups = kInPad / 4, kEach = (R * kGroups + kRowThreads - 1) / kRowThreads;
    static_assert(kIn % 4 == 0, "a row is whole groups of 4");
    f32x4 v[kEach];
#pragma unroll
    for (int i = 0; i < kEach; ++i) {
        const int t = threadIdx.x + i * kRowThreads, m = t / kGroups, k = 4 * (t - m * kGroups);
        v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (m < R && m0 + m < B && k < kIn)
            v[i] = *reinterpret_cast<const f32x4u*>(X + (size_t)(m0 + m) * kIn + k);
    }
#pragma unroll
    for (int i = 0; i < kEach; ++i) {
        const int t = threadIdx.x + i * kRowThreads, m = t / kGroups, k = 4 * (t - m * kGroups);
        if (m < R)
            *reinterpret_cast<uint2*>(s_in + m * kLdIn + k) =
                make_uint2(f2bf(v[i].x) | ((uint32_t)f2bf(v[i].y) << 16),
                           f2bf(v[i].z) | ((uint32_t)f2bf(v[i].w) << 16));
    }
}

// Hidden layer l: s_out = relu(s_in W^T + b) in BF16.
template <int RT, int NK>
__device__ __forceinline__ void hidden_layer(const MlpDev& d, int l, const uint16_t* s_in, int lda,
                                             const Frags<NK>& f, uint16_t* s_out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float* bias = d.params + d.off_b[l] + 32 * wave + (lane & 15);
    const float b0 = bias[0], b1 = bias[16];
    f32x4 acc[2][RT];
    rows_product<RT, NK>(s_in, lda, f, acc);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int n = (2 * wave + j) * 16 + (lane & 15);
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                s_out[(16 * i + 4 * (lane >> 4) + r) * kLdHid + n] =
                    f2bf(fmaxf(acc[j][i][r] + (j ? b1 : b0), 0.0f));
    }
}

constexpr int kHidTiles = kHidden / 16, kOutTiles = kOutPad / 16;
constexpr int kNkIn = kInPad / 32, kNkHid = kHidden / 32, kNkOut = kOutPad / 32;

template <int RT>
__global__ __launch_bounds__(kRowThreads, 2) void k_mlp_forward(MlpDev d, const float* __restrict__ X,
                                                            int B, float* __restrict__ out, int ld,
                                                            int n_out, int rows) {
    constexpr int R = 16 * RT;
    __shared__ __align__(16) uint16_t s_in[R * kLdIn];
    __shared__ __align__(16) uint16_t s_a[R * kLdHid], s_b[R * kLdHid];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m0 = blockIdx.x * R;
    uint16_t *in = s_a, *next = s_b;
    Frags<kNkHid> f;
    {
        Frags<kNkIn> f0;
        load_frags(d.Wb[0], kHidTiles, f0);
        load_rows<R>(X, B, m0, s_in);
        load_frags(d.Wb[1], kHidTiles, f);
        __syncthreads();
        hidden_layer<RT>(d, 0, s_in, kLdIn, f0, in);
        __syncthreads();
    }
#pragma unroll 1
    for (int l = 1; l < 4; ++l) {
        Frags<kNkHid> ahead;
        load_frags(d.Wb[l + 1], l < 3 ? kHidTiles : kOutTiles, ahead);
        hidden_layer<RT>(d, l, in, kLdHid, f, next);
        __syncthreads();
        uint16_t* u = in;
        in = next;
        next = u;
        f = ahead;
    }
    if (2 * wave >= kOutTiles) return;
    f32x4 acc[2][RT];
    rows_product<RT>(in, kLdHid, f, acc);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int n = (2 * wave + j) * 16 + (lane & 15);
        if (n >= n_out) continue;
        const float bias = n < kOut ? d.params[d.off_b[4] + n] : 0.0f;
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + 16 * i + 4 * (lane >> 4) + r;
                if (m < rows) out[(size_t)m * ld + n] = acc[j][i][r] + bias;
            }
    }
}

// A workgroup takes a CU (its weights in registers).  As long as every 16 rows
// have one of the 256 CUs, up to 4096 rows, a workgroup takes 16 (2048 to 4096
// rows: 13.5 to 14.7 us; 4096 rows by 32: 18.6); beyond that 32, in one pass over
// the CUs where 16 would need two (4999 rows 19 us, 8192: 20 to 25).
constexpr int kNarrowRows = 16 * 256;

void launch_mlp_forward(hipStream_t s, const MlpDev& d, const float* X, int B, float* out, int ld,
                        int n_out, int rows) {
    if (B > kNarrowRows)
        k_mlp_forward<2><<<(rows + 31) / 32, kRowThreads, 0, s>>>(d, X, B, out, ld, n_out, rows);
    else
        k_mlp_forward<1><<<(rows + 15) / 16, kRowThreads, 0, s>>>(d, X, B, out, ld, n_out, rows);
}

// Column c of 16 BF16 rows in LDS to batch rows m0 .. of dst, in fragment order.
__device__ __forceinline__ void store_column(const uint16_t* s, int ld, int c, uint16_t* dst, int m0,
                                             int Bp) {
    uint32_t w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
        w[i] = (uint32_t)s[(2 * i) * ld + c] | ((uint32_t)s[(2 * i + 1) * ld + c] << 16);
    uint4* q = reinterpret_cast<uint4*>(dst + frag_at(c, m0, Bp / 32));
    q[0] = make_uint4(w[0], w[1], w[2], w[3]);
    q[16] = make_uint4(w[4], w[5], w[6], w[7]);
}

// Mixture NLL of 16 rows and its gradient with respect to the outputs, in
// place (thread = row * 16 + component, threads 0 .. 255; the workgroup calls
// it).  Outputs: logits [16], means [16][6], log-std [16][6] clamped to
// [-4, 2].  Sums over the components run in their order.  Rows past the batch
// get zeros; s_loss the rows' losses.
__device__ __forceinline__ void mixture_nll_rows(float* s_y, const float* __restrict__ Z, int B, int m0,
                                                 float* s_loss) {
    const int m = threadIdx.x >> 4, k = threadIdx.x & 15;
    float gk = 0.0f, gm[kDState], gs[kDState];
    for (int e = 0; e < kDState; ++e) gm[e] = gs[e] = 0.0f;
    float loss = 0.0f;
    const bool row = threadIdx.x < 256, real = row && m0 + m < B;
    if (real) {   // (whole 16-lane groups)
        const float* y = s_y + m * kLdOut;
        auto max16 = [&](float v) {
            for (int o = 8; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 16));
            return v;
        };
        auto sum16 = [&](float v) {
            float s = 0.0f;
            for (int i = 0; i < kComp; ++i) s += __shfl(v, i, 16);
            return s;
        };
        float z[kDState];
        for (int e = 0; e < kDState; ++e) z[e] = Z[(size_t)(m0 + m) * kDState + e];
        const float yk = y[k];
        const float lmax = max16(yk);
        const float lse_logit = lmax + logf(sum16(expf(yk - lmax)));
        float q = 0.0f, ssum = 0.0f;
        for (int e = 0; e < kDState; ++e) {
            const float sd = fminf(fmaxf(y[kComp * 7 + k * kDState + e], kLogStdMin), kLogStdMax);
            const float rr = (z[e] - y[kComp + k * kDState + e]) * expf(-sd);
            q += rr * rr;
            ssum += sd;
        }
        const float a = (yk - lse_logit) - 0.5f * q - ssum - 0.5f * kDState * 1.8378770664093453f;
        const float amax = max16(a);
        const float lse_a = amax + logf(sum16(expf(a - amax)));
        loss = -lse_a;
        const float invB = 1.0f / (float)B;
        const float w = expf(a - lse_a);
        const float pi = expf(yk - lse_logit);
        gk = (pi - w) * invB;
        for (int e = 0; e < kDState; ++e) {
            const float raw = y[kComp * 7 + k * kDState + e];
            const float sd = fminf(fmaxf(raw, kLogStdMin), kLogStdMax);
            const float inv = expf(-sd);
            const float rr = (z[e] - y[kComp + k * kDState + e]) * inv;
            gm[e] = -w * rr * inv * invB;
            const bool inside = raw > kLogStdMin && raw < kLogStdMax;
            gs[e] = inside ? w * (1.0f - rr * rr) * invB : 0.0f;
        }
    }
    __syncthreads();   // every output read
    if (row) {
        float* g = s_y + m * kLdOut;
        g[k] = gk;
        for (int e = 0; e < kDState; ++e) {
            g[kComp + k * kDState + e] = gm[e];
            g[kComp * 7 + k * kDState + e] = gs[e];
        }
        g[kOut + k] = 0.0f;   // (the padding columns)
        if (k == 0) s_loss[m] = loss;
    }
    __syncthreads();
}

// Gradient of layer l's inputs (masked by their ReLU: s_h, the layer's input
// activations) from its output gradients in s_g, which it replaces; partials
// of layer l - 1's bias gradient and its output gradients, batch rows
// contiguous, to memory.
template <int NK>
__device__ __forceinline__ void back_layer(const MlpDev& d, int l, uint16_t* s_g, const uint16_t* s_h,
                                           const Frags<NK>& f, float* bpart, int m0, int Bp) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    f32x4 acc[2][1];
    rows_product<1>(s_g, kLdHid, f, acc);
    __syncthreads();   // every gradient read
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int n = (2 * wave + j) * 16 + (lane & 15);
        float sum = 0.0f;
        uint32_t h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 4 * (lane >> 4) + r;
            const float v = acc[j][0][r] * (bf2f(s_h[m * kLdHid + n]) > 0.0f ? 1.0f : 0.0f);
            sum += v;
            h[r] = f2bf(v);
            s_g[m * kLdHid + n] = (uint16_t)h[r];
        }
        *reinterpret_cast<uint2*>(d.GT[l - 1] + frag_at(n, m0 + 4 * (lane >> 4), Bp / 32)) =
            make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
        sum += __shfl_xor(sum, 16, 64);
        sum += __shfl_xor(sum, 32, 64);
        if (lane < 16) bpart[(l - 1) * kHidden + n] = sum;
    }
    __syncthreads();
}

__global__ __launch_bounds__(kRowThreads, 2) void k_mlp_rows(MlpDev d, const float* __restrict__ X,
                                                         const float* __restrict__ Z, int B, int Bp) {
    // the input rows' LDS holds the outputs, then their gradients, in FP32
    __shared__ __align__(16) float s_y[16 * kLdOut];
    static_assert(16 * kLdOut * 4 >= 16 * kLdIn * 2, "the input rows fit");
    __shared__ __align__(16) uint16_t s_h[4][16 * kLdHid];
    __shared__ __align__(16) uint16_t s_g[16 * kLdHid];
    __shared__ float s_loss[16];
    uint16_t* s_in = reinterpret_cast<uint16_t*>(s_y);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int m0 = blockIdx.x * 16;
    Frags<kNkIn> f0;
    Frags<kNkHid> f1, f2;
    load_frags(d.Wb[0], kHidTiles, f0);
    load_rows<16>(X, B, m0, s_in);
    load_frags(d.Wb[1], kHidTiles, f1);
    __syncthreads();
    hidden_layer<1>(d, 0, s_in, kLdIn, f0, s_h[0]);
    load_frags(d.Wb[2], kHidTiles, f2);
    if (t < kInPad) store_column(s_in, kLdIn, t, d.HT[0], m0, Bp);
    __syncthreads();
    hidden_layer<1>(d, 1, s_h[0], kLdHid, f1, s_h[1]);
    load_frags(d.Wb[3], kHidTiles, f1);
    __syncthreads();
    hidden_layer<1>(d, 2, s_h[1], kLdHid, f2, s_h[2]);
    load_frags(d.Wb[4], kOutTiles, f2);
    __syncthreads();
    hidden_layer<1>(d, 3, s_h[2], kLdHid, f1, s_h[3]);
    Frags<kNkOut> g4;
    load_frags(d.WbT[4], kHidTiles, g4);
    __syncthreads();
    if (2 * wave < kOutTiles) {
        f32x4 acc[2][1];
        rows_product<1>(s_h[3], kLdHid, f2, acc);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = (2 * wave + j) * 16 + (lane & 15);
            const float bias = n < kOut ? d.params[d.off_b[4] + n] : 0.0f;
#pragma unroll
            for (int r = 0; r < 4; ++r) s_y[(4 * (lane >> 4) + r) * kLdOut + n] = acc[j][0][r] + bias;
        }
    }
    load_frags(d.WbT[3], kHidTiles, f1);
    // the layer inputs' columns go out while the losses are taken
    if (t >= 256) {
#pragma unroll
        for (int l = 1; l < 5; ++l)
            store_column(s_h[l - 1], kLdHid, t - 256, d.HT[l], m0, Bp);
    }
    __syncthreads();
    mixture_nll_rows(s_y, Z, B, m0, s_loss);
    float* bpart = d.bpart + (size_t)blockIdx.x * kBiasTotal;
    if (t == 0) {
        float s = 0.0f;
        for (int m = 0; m < 16; ++m) s += s_loss[m];
        d.lpart[blockIdx.x] = s;
    }
    if (t < kOutPad) {
        float s = 0.0f;
        uint32_t h[16];
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const float v = s_y[m * kLdOut + t];
            s += v;
            h[m] = f2bf(v);
            s_g[m * kLdHid + t] = (uint16_t)h[m];
        }
        if (t < kOut) bpart[4 * kHidden + t] = s;
        uint4* g = reinterpret_cast<uint4*>(d.GT[4] + frag_at(t, m0, Bp / 32));
        g[0] = make_uint4(h[0] | h[1] << 16, h[2] | h[3] << 16, h[4] | h[5] << 16, h[6] | h[7] << 16);
        g[16] = make_uint4(h[8] | h[9] << 16, h[10] | h[11] << 16, h[12] | h[13] << 16, h[14] | h[15] << 16);
    }
    __syncthreads();
    back_layer(d, 4, s_g, s_h[3], g4, bpart, m0, Bp);
    load_frags(d.WbT[2], kHidTiles, f2);
    back_layer(d, 3, s_g, s_h[2], f1, bpart, m0, Bp);
    load_frags(d.WbT[1], kHidTiles, f1);
    back_layer(d, 2, s_g, s_h[1], f2, bpart, m0, Bp);
    back_layer(d, 1, s_g, s_h[0], f1, bpart, m0, Bp);
}

// ---------------------------------------------------------------------------
// Weight gradients of every layer in one launch: G^T H, both with the batch
// rows contiguous, a workgroup a 16 x 128 tile (a wave 16 x 32 of it); then
// workgroups for the bias gradients (64 entries each) and one for the mean
// loss.  An element is one chain of products over the batch rows in order
// (kept: split sums of the rows moved the weights by some 1e-7 and with it a
// few of their BF16 roundings a step).  The chain is as long as the
// batch, so eight products' operands are in flight while eight are taken.
// ---------------------------------------------------------------------------
constexpr int wgrad_cols(int l) { return (mlp_in_p(l) + 127) / 128; }
constexpr int tiles_of(int l) { return (mlp_out_p(l) / 16) * wgrad_cols(l); }
constexpr int kWgradTiles = tiles_of(0) + tiles_of(1) + tiles_of(2) + tiles_of(3) + tiles_of(4);
constexpr int kBiasBlocks = (kBiasTotal + 63) / 64;

__global__ __launch_bounds__(256, 1) void k_mlp_wgrad(MlpDev d, int Bp, int B, float* __restrict__ loss) {
    __shared__ double s_sum[256];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    int bx = blockIdx.x;
    if (bx < kWgradTiles) {
        int l = 0;
        while (bx >= tiles_of(l)) bx -= tiles_of(l++);
        const int tn = wgrad_cols(l);
        const int m0 = (bx / tn) * 16, n0 = (bx % tn) * 128 + wave * 32;
        if (n0 >= mlp_in_p(l)) return;
        const int r = lane & 15, nk = Bp / 32;
        const bf16x8* A = reinterpret_cast<const bf16x8*>(d.GT[l]) + (size_t)(m0 / 16) * nk * 64 + lane;
        const bf16x8* B0 = reinterpret_cast<const bf16x8*>(d.HT[l]) + (size_t)(n0 / 16) * nk * 64 + lane;
        const bf16x8* B1 = B0 + (size_t)nk * 64;
        constexpr int kAhead = 8;
        bf16x8 cur[kAhead][3], nxt[kAhead][3];
        auto load = [&](bf16x8 (&v)[kAhead][3], int k0) {
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int k = 64 * min(k0 + u, nk - 1);
                v[u][0] = A[k];
                v[u][1] = B0[k];
                v[u][2] = B1[k];
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
        auto take = [&](const bf16x8 (&v)[kAhead][3], int k0) {
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
                if (k0 + u < nk) {
                    acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v[u][0], v[u][1], acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v[u][0], v[u][2], acc[1], 0, 0, 0);
                }
        };
        load(cur, 0);
        for (int k = 0; k < nk; k += 2 * kAhead) {
            load(nxt, k + kAhead);
            take(cur, k);
            load(cur, k + 2 * kAhead);
            take(nxt, k + kAhead);
        }
        float* W = d.grads + d.off_W[l];
        const int in = mlp_in(l), out = mlp_out(l);
        for (int j = 0; j < 2; ++j)
            for (int rr = 0; rr < 4; ++rr) {
                const int m = m0 + 4 * (lane >> 4) + rr, n = n0 + 16 * j + r;
                if (m < out && n < in) W[(size_t)m * in + n] = acc[j][rr];
            }
        return;
    }
    bx -= kWgradTiles;
    const int nblk = Bp / 16;
    if (bx < kBiasBlocks) {
        // entry e over the row blocks w, w + 4, ..., the four sums joined in order
        const int e = bx * 64 + lane;
        double s = 0.0;
        if (e < kBiasTotal) {
#pragma unroll 8
            for (int b = wave; b < nblk; b += 4) s += (double)d.bpart[(size_t)b * kBiasTotal + e];
        }
        s_sum[t] = s;
        __syncthreads();
        if (wave == 0 && e < kBiasTotal) {
            const int l = min(e / kHidden, kLayers - 1);
            d.grads[d.off_b[l] + e - l * kHidden] =
                (float)(((s_sum[lane] + s_sum[64 + lane]) + s_sum[128 + lane]) + s_sum[192 + lane]);
        }
        return;
    }
    double s = 0.0;
    for (int b = t; b < nblk; b += 256) s += (double)d.lpart[b];
    s_sum[t] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w) s_sum[t] += s_sum[t + w];
        __syncthreads();
    }
    if (t == 0) *loss = (float)(s_sum[0] / (double)B);
}

void launch_mlp_grad(hipStream_t s, const MlpDev& d, const float* X, const float* Z, int B, int Bp,
                     float* loss) {
    k_mlp_rows<<<Bp / 16, kRowThreads, 0, s>>>(d, X, Z, B, Bp);
    k_mlp_wgrad<<<kWgradTiles + kBiasBlocks + 1, 256, 0, s>>>(d, Bp, B, loss);
}

// Layer of parameter i, and whether it is a weight.
__device__ __forceinline__ int layer_of(const MlpDev& d, int i, bool& weight) {
    int l = 0;
    while (l < kLayers - 1 && i >= d.off_W[l + 1]) ++l;
    weight = i < d.off_b[l];
    return l;
}

__device__ __forceinline__ void store_weight(const MlpDev& d, int l, int i, float w) {
    const int e = i - d.off_W[l], n = e / mlp_in(l), k = e - n * mlp_in(l);
    const uint16_t h = f2bf(w);
    d.Wb[l][frag_at(n, k, mlp_in_p(l) / 32)] = h;
    d.WbT[l][frag_at(k, n, mlp_out_p(l) / 32)] = h;
}

// ---------------------------------------------------------------------------
// Adam (Kingma & Ba) on the FP32 master parameters, and the BF16 copies of the
// weights it changes.
// ---------------------------------------------------------------------------
// (1 - beta) is passed rounded from its exact value: 1 - 0.999f in FP32 would be
// 1.3e-5 relatively off 0.001.
__global__ __launch_bounds__(256) void k_adam(MlpDev d, float lr, float b1, float b2,
                                              float omb1, float omb2, float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= d.n_params) return;
    bool weight;
    const int l = layer_of(d, i, weight);
    const float gi = d.grads[i];
    const float a = b1 * d.m1[i] + omb1 * gi;
    const float b = b2 * d.m2[i] + omb2 * gi * gi;
    d.m1[i] = a;
    d.m2[i] = b;
    const float p = d.params[i] - lr * (a / c1) / (sqrtf(b / c2) + eps);
    d.params[i] = p;
    if (weight) store_weight(d, l, i, p);
}

void launch_adam(hipStream_t s, const MlpDev& d, float lr, int t) {
    const double b1 = 0.9, b2 = 0.999;
    const float c1 = (float)(1.0 - pow(b1, t)), c2 = (float)(1.0 - pow(b2, t));
    k_adam<<<(d.n_params + 255) / 256, 256, 0, s>>>(d, lr, (float)b1, (float)b2, (float)(1.0 - b1),
                                                    (float)(1.0 - b2), 1e-8f, c1, c2);
}

// BF16 weights of every layer (a workgroup row per layer), zero padded.
__global__ __launch_bounds__(256) void k_refresh_bf16(MlpDev d) {
    const int l = blockIdx.y;
    const int in = mlp_in(l), out = mlp_out(l), in_p = mlp_in_p(l), out_p = mlp_out_p(l);
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= out_p * in_p) return;
    const int n = t / in_p, k = t - n * in_p;
    const uint16_t h = (n < out && k < in) ? f2bf(d.params[d.off_W[l] + (size_t)n * in + k]) : (uint16_t)0;
    d.Wb[l][frag_at(n, k, in_p / 32)] = h;
    d.WbT[l][frag_at(k, n, out_p / 32)] = h;
}

void launch_refresh_bf16(hipStream_t s, const MlpDev& d) {
    k_refresh_bf16<<<dim3((kHidden * kInPad + 255) / 256, kLayers), 256, 0, s>>>(d);
}

// ---------------------------------------------------------------------------
// Condition vectors: start (6), goal centre (3) and half-size (3), then up to
// 64 boxes (lo xyz, hi xyz), zero padded.
// ---------------------------------------------------------------------------
__global__ void k_condition(const float* __restrict__ x_init, const float* __restrict__ goal,
                            const float* __restrict__ boxes, const int32_t* __restrict__ n_obs,
                            int q, int max_boxes_in, float* __restrict__ cond) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= q * kIn) return;
    const int i = t / kIn, j = t - i * kIn;
    float v = 0.0f;
    if (j < 6) {
        v = x_init[(size_t)i * 6 + j];
    } else if (j < 9) {
        v = 0.5f * (goal[(size_t)i * 6 + (j - 6)] + goal[(size_t)i * 6 + 3 + (j - 6)]);
    } else if (j < 12) {
        v = 0.5f * (goal[(size_t)i * 6 + 3 + (j - 9)] - goal[(size_t)i * 6 + (j - 9)]);
    } else {
        const int b = (j - 12) / 6, c = (j - 12) % 6;
        if (b < n_obs[i] && b < kMaxBoxes) v = boxes[((size_t)i * max_boxes_in + b) * 6 + c];
    }
    cond[(size_t)i * kIn + j] = v;
}

void launch_condition(hipStream_t s, const float* x_init, const float* goal, const float* boxes,
                      const int32_t* n_obs, int q, int max_boxes_in, float* cond) {
    const int n = q * kIn;
    k_condition<<<(n + 255) / 256, 256, 0, s>>>(x_init, goal, boxes, n_obs, q, max_boxes_in, cond);
}

// ---------------------------------------------------------------------------
// Mixture sampling: one draw per thread, workgroups of one query each.  The
// component is chosen by the inverse CDF of softmax(logits) at u * total
// (FP64), the state is mu + sigma * eps, clamped to the state box.  The CDF and
// the sigmas (112 FP64 exponentials) are the query's and taken once a
// workgroup; taken by every draw they were most of the kernel.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_sample(const float* __restrict__ Y, int ldy, int n, int per_q,
                                                const float* __restrict__ u,
                                                const float* __restrict__ eps,
                                                float* __restrict__ out) {
    __shared__ double s_e[kComp], s_cdf[kComp], s_mu[kComp * kDState], s_sd[kComp * kDState];
    const int i = blockIdx.x / per_q;
    const float* y = Y + (size_t)i * ldy;
    const int t = threadIdx.x;
    if (t < kComp * kDState) {
        s_mu[t] = (double)y[kComp + t];
        s_sd[t] = exp(fmin(fmax((double)y[kComp * 7 + t], (double)kLogStdMin), (double)kLogStdMax));
    } else if (t >= 128 && t < 128 + kComp) {
        double mx = -INFINITY;
        for (int k = 0; k < kComp; ++k) mx = fmax(mx, (double)y[k]);
        s_e[t - 128] = exp((double)y[t - 128] - mx);
    }
    __syncthreads();
    if (t == 0) {
        double acc = 0.0;
        for (int k = 0; k < kComp; ++k) {
            acc += s_e[k];
            s_cdf[k] = acc;
        }
    }
    __syncthreads();
    const int j = (blockIdx.x - i * per_q) * 256 + t;
    if (j >= n) return;
    const size_t d = (size_t)i * n + j;
    const double target = (double)u[d] * s_cdf[kComp - 1];
    int k = 0;
    while (k < kComp - 1 && !(target < s_cdf[k])) ++k;
    for (int e = 0; e < kDState; ++e) {
        double v = s_mu[k * kDState + e] + s_sd[k * kDState + e] * (double)eps[d * kDState + e];
        v = fmin(fmax(v, e < 3 ? 0.0 : -0.5), e < 3 ? 1.0 : 0.5);
        out[d * kDState + e] = (float)v;
    }
}

void launch_sample(hipStream_t s, const float* Y, int ldy, int q, int n, const float* u,
                   const float* eps, float* out) {
    const int per_q = (n + 255) / 256;
    k_sample<<<q * per_q, 256, 0, s>>>(Y, ldy, n, per_q, u, eps, out);
}

}  // namespace pump
