// Per-query setup operations: the particle deviation table and BuildGraph
// (Alg. 3), shared by the single-query kernels and the batched engine.
#pragma once

#include "box_bins.hpp"
#include "device_math.hpp"
#include "pump_internal.hpp"

namespace pump {


// ---------------------------------------------------------------------------
// Particle deviation table (Sec. III-B particles; eq. (2) closed loop).
// Per (axis a, particle j) the recurrence
//   dx_{s+1} = A_cl dx_s + L (xi[s][2a][j], xi[s][2a+1][j])^T,  dx_0 = 0
// runs in FP64 and the position part D[s][a][j] is stored in FP32.  The
// steps are cut into chunks of kDevChunk so that many lanes work at once:
// (1) every (chunk, a, j) runs its chunk from a zero state, giving the
// chunk's own response E_k; (2) every (a, j) chains the chunk start states,
// X_{k+1} = A_cl^C X_k + E_k; (3) every (chunk, a, j) reruns its chunk from
// X_k and stores D.  The state at a chunk start differs from the sequential
// recurrence only by FP64 rounding.
// Scratch: E and X0, each [K][3][N] double2 with K = ceil(S / kDevChunk).
// ---------------------------------------------------------------------------
constexpr int kDevChunk = 16;

struct DevCoef {
    double a00, a01, a10, a11, l00, l10, l11;
};

__device__ __forceinline__ void dev_run_chunk(const float* __restrict__ noise, int N, int S, int a,
                                              int j, int k, const DevCoef& m, double& p,
                                              double& v, float* __restrict__ D) {
    const int s0 = k * kDevChunk;
    float w0[kDevChunk], w1[kDevChunk];
#pragma unroll
    for (int u = 0; u < kDevChunk; ++u) {
        const int s = s0 + u < S ? s0 + u : S - 1;
        w0[u] = noise[((size_t)s * 6 + 2 * a) * N + j];
        w1[u] = noise[((size_t)s * 6 + 2 * a + 1) * N + j];
    }
#pragma unroll
    for (int u = 0; u < kDevChunk; ++u) {
        if (s0 + u >= S) break;
        const double pn = m.a00 * p + m.a01 * v + m.l00 * (double)w0[u];
        const double vn = m.a10 * p + m.a11 * v + (m.l10 * (double)w0[u] + m.l11 * (double)w1[u]);
        p = pn;
        v = vn;
        if (D) D[((size_t)(s0 + u + 1) * 3 + a) * N + j] = (float)p;
    }
}

// (1) chunk responses; thread t = (k * 3 + a) * N + j
__device__ __forceinline__ void dev_local_dev(const float* __restrict__ noise, double* __restrict__ E,
                                              int N, int S, const DevCoef& m) {
    const int K = (S + kDevChunk - 1) / kDevChunk;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= K * 3 * N) return;
    const int j = t % N, a = (t / N) % 3, k = t / (3 * N);
    double p = 0.0, v = 0.0;
    dev_run_chunk(noise, N, S, a, j, k, m, p, v, nullptr);
    E[2 * (size_t)t] = p;
    E[2 * (size_t)t + 1] = v;
}

// (2) chunk start states; thread col = a * N + j
__device__ __forceinline__ void dev_carry_dev(const double* __restrict__ E, double* __restrict__ X0,
                                              int N, int S, const DevCoef& m) {
    const int K = (S + kDevChunk - 1) / kDevChunk;
    const int col = blockIdx.x * blockDim.x + threadIdx.x;
    if (col >= 3 * N) return;
    // Phi = A_cl^C
    double f00 = 1.0, f01 = 0.0, f10 = 0.0, f11 = 1.0;
    for (int u = 0; u < kDevChunk; ++u) {
        const double g00 = m.a00 * f00 + m.a01 * f10, g01 = m.a00 * f01 + m.a01 * f11;
        const double g10 = m.a10 * f00 + m.a11 * f10, g11 = m.a10 * f01 + m.a11 * f11;
        f00 = g00; f01 = g01; f10 = g10; f11 = g11;
    }
    double p = 0.0, v = 0.0;
    for (int k = 0; k < K; ++k) {
        const size_t t = (size_t)k * 3 * N + col;
        X0[2 * t] = p;
        X0[2 * t + 1] = v;
        const double pn = f00 * p + f01 * v + E[2 * t];
        const double vn = f10 * p + f11 * v + E[2 * t + 1];
        p = pn;
        v = vn;
    }
}

// (3) the table; thread t = (k * 3 + a) * N + j
__device__ __forceinline__ void dev_final_dev(const float* __restrict__ noise, const double* __restrict__ X0,
                                              float* __restrict__ D, int N, int S, const DevCoef& m) {
    const int K = (S + kDevChunk - 1) / kDevChunk;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= K * 3 * N) return;
    const int j = t % N, a = (t / N) % 3, k = t / (3 * N);
    if (k == 0) D[(size_t)a * N + j] = 0.0f;
    double p = X0[2 * (size_t)t], v = X0[2 * (size_t)t + 1];
    dev_run_chunk(noise, N, S, a, j, k, m, p, v, D);
}

// ---------------------------------------------------------------------------
// The deviation table under LQG tracking.  Per (axis a, particle j) the
// joint state z = (dp, dv, p_hat, v_hat) follows z' = m z + e xi with
// xi = (noise[s][2a][j], noise[s][2a+1][j], noise_meas[s][a][j]), z_0 = 0;
// D stores dp.  Same three chunked passes as above with a 4-state carry
// (Phi = m^C).  Scratch: E and X0, each [K][3][N] of 4 doubles.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void lqg_run_chunk(const float* __restrict__ noise,
                                              const float* __restrict__ meas, int N, int S, int a,
                                              int j, int k, const LqgCoef& q, double z[4],
                                              float* __restrict__ D) {
    const int s0 = k * kDevChunk;
    float w0[kDevChunk], w1[kDevChunk], w2[kDevChunk];
#pragma unroll
    for (int u = 0; u < kDevChunk; ++u) {
        const int s = s0 + u < S ? s0 + u : S - 1;
        w0[u] = noise[((size_t)s * 6 + 2 * a) * N + j];
        w1[u] = noise[((size_t)s * 6 + 2 * a + 1) * N + j];
        w2[u] = meas[((size_t)s * 3 + a) * N + j];
    }
#pragma unroll
    for (int u = 0; u < kDevChunk; ++u) {
        if (s0 + u >= S) break;
        lqg_step(q, z, (double)w0[u], (double)w1[u], (double)w2[u]);
        if (D) D[((size_t)(s0 + u + 1) * 3 + a) * N + j] = (float)z[0];
    }
}

// (1) chunk responses; thread t = (k * 3 + a) * N + j
__device__ __forceinline__ void lqg_local_dev(const float* __restrict__ noise,
                                              const float* __restrict__ meas,
                                              double* __restrict__ E, int N, int S,
                                              const LqgCoef& q) {
    const int K = (S + kDevChunk - 1) / kDevChunk;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= K * 3 * N) return;
    const int j = t % N, a = (t / N) % 3, k = t / (3 * N);
    double z[4] = {0.0, 0.0, 0.0, 0.0};
    lqg_run_chunk(noise, meas, N, S, a, j, k, q, z, nullptr);
#pragma unroll
    for (int i = 0; i < 4; ++i) E[4 * (size_t)t + i] = z[i];
}

// (2) chunk start states; thread col = a * N + j
__device__ __forceinline__ void lqg_carry_dev(const double* __restrict__ E,
                                              double* __restrict__ X0, int N, int S,
                                              const LqgCoef& q) {
    const int K = (S + kDevChunk - 1) / kDevChunk;
    const int col = blockIdx.x * blockDim.x + threadIdx.x;
    if (col >= 3 * N) return;
    double f[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) f[i] = (i % 5 == 0) ? 1.0 : 0.0;
    for (int u = 0; u < kDevChunk; ++u) {
        double g[16];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                g[4 * i + c] = q.m[4 * i] * f[c] + q.m[4 * i + 1] * f[4 + c] +
                               q.m[4 * i + 2] * f[8 + c] + q.m[4 * i + 3] * f[12 + c];
#pragma unroll
        for (int i = 0; i < 16; ++i) f[i] = g[i];
    }
    double z[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k = 0; k < K; ++k) {
        const size_t t = (size_t)k * 3 * N + col;
        double zn[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            X0[4 * t + i] = z[i];
            zn[i] = f[4 * i] * z[0] + f[4 * i + 1] * z[1] + f[4 * i + 2] * z[2] +
                    f[4 * i + 3] * z[3] + E[4 * t + i];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) z[i] = zn[i];
    }
}

// (3) the table; thread t = (k * 3 + a) * N + j
__device__ __forceinline__ void lqg_final_dev(const float* __restrict__ noise,
                                              const float* __restrict__ meas,
                                              const double* __restrict__ X0,
                                              float* __restrict__ D, int N, int S,
                                              const LqgCoef& q) {
    const int K = (S + kDevChunk - 1) / kDevChunk;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= K * 3 * N) return;
    const int j = t % N, a = (t / N) % 3, k = t / (3 * N);
    if (k == 0) D[(size_t)a * N + j] = 0.0f;
    double z[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) z[i] = X0[4 * (size_t)t + i];
    lqg_run_chunk(noise, meas, N, S, a, j, k, q, z, D);
}

// Bounding box of the particle cloud at each step: cloud[s] = (min_j D[s][a][j], max_j ...).
__device__ __forceinline__ void cloud_dev(const float* __restrict__ D, float* __restrict__ cloud, int N) {
    __shared__ float smin[3][256], smax[3][256];
    int s = blockIdx.x, t = threadIdx.x;
    for (int a = 0; a < 3; ++a) {
        float mn = INFINITY, mx = -INFINITY;
        for (int j = t; j < N; j += blockDim.x) {
            float d = D[((size_t)s * 3 + a) * N + j];
            mn = fminf(mn, d);
            mx = fmaxf(mx, d);
        }
        smin[a][t] = mn;
        smax[a][t] = mx;
    }
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if (t < w)
            for (int a = 0; a < 3; ++a) {
                smin[a][t] = fminf(smin[a][t], smin[a][t + w]);
                smax[a][t] = fmaxf(smax[a][t], smax[a][t + w]);
            }
        __syncthreads();
    }
    if (t < 3) {
        cloud[(size_t)s * 6 + t] = smin[t][0];
        cloud[(size_t)s * 6 + 3 + t] = smax[t][0];
    }
}

__device__ __forceinline__ void gcloud_dev(const float* __restrict__ cloud, float* __restrict__ g, int S1) {
    __shared__ float sm[6][256];
    const int t = threadIdx.x;
    float v[6];
    for (int k = 0; k < 6; ++k) v[k] = k < 3 ? INFINITY : -INFINITY;
    for (int s = t; s < S1; s += blockDim.x)
        for (int k = 0; k < 6; ++k) {
            float c = cloud[(size_t)s * 6 + k];
            v[k] = k < 3 ? fminf(v[k], c) : fmaxf(v[k], c);
        }
    for (int k = 0; k < 6; ++k) sm[k][t] = v[k];
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if (t < w)
            for (int k = 0; k < 6; ++k)
                sm[k][t] = k < 3 ? fminf(sm[k][t], sm[k][t + w]) : fmaxf(sm[k][t], sm[k][t + w]);
        __syncthreads();
    }
    if (t < 6) g[t] = sm[t][0];
}

// ---------------------------------------------------------------------------
// Node validity (sample not in a closed obstacle box) and goal membership
// (position in the closed goal box).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void mark_valid_dev(const float* __restrict__ X, int n, const float* __restrict__ obs,
                             int n_obs, float g0, float g1, float g2, float g3, float g4, float g5,
                             uint8_t* __restrict__ valid, uint8_t* __restrict__ goal,
                             int32_t* __restrict__ bad) {
    int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n_obs) {
        // obstacle sanity: finite, ordered, inside [-16, 16]
        const float* b = obs + (size_t)v * 6;
        bool okb = true;
        for (int k = 0; k < 3; ++k)
            okb &= (b[k] <= b[3 + k]) & (fabsf(b[k]) <= 16.0f) & (fabsf(b[3 + k]) <= 16.0f);
        if (!okb) atomicOr(bad, 1);
    }
    if (v >= n) return;
    float p0 = X[(size_t)v * 6], p1 = X[(size_t)v * 6 + 1], p2 = X[(size_t)v * 6 + 2];
    if (!(fabsf(p0) <= 16.0f && fabsf(p1) <= 16.0f && fabsf(p2) <= 16.0f)) atomicOr(bad, 1);
    bool in = false;
    for (int o = 0; o < n_obs; ++o) {
        const float* b = obs + (size_t)o * 6;
        in |= (p0 >= b[0]) & (p0 <= b[3]) & (p1 >= b[1]) & (p1 <= b[4]) & (p2 >= b[2]) & (p2 <= b[5]);
    }
    if (v == 0 && in) atomicOr(bad, 2);
    valid[v] = in ? 0 : 1;
    bool g = (p0 >= g0) & (p0 <= g3) & (p1 >= g1) & (p1 <= g4) & (p2 >= g2) & (p2 <= g5);
    goal[v] = (!in && g) ? 1 : 0;
}

// ---------------------------------------------------------------------------
// BuildGraph (Alg. 3).  Edge v -> u iff both nodes are valid, u != v,
// c*(v,u) < r_n, tau* > 1e-6 and the nominal trajectory meets no obstacle
// (continuous, exact; closed boxes).  The result is a bit matrix (row v,
// bit u) and per-row counts; after a scan of the counts, pass 2 writes each
// row's neighbours in ascending order with their (tau*, c*).
//
// Pass 1 runs as stages, each its own kernel so that the register-heavy
// exact box test does not hold down the occupancy of the others:
//   near    a workgroup per kNearRows rows: every target through the Near
//           rejection test, the survivors steered densely (tau*, c*); near
//           connections -> the near list;
//   boxes   each near connection's pieces against the boxes in their bins; a
//           proved hit blocks it, an unsure (connection, box) goes to the exact
//           queue; connections not blocked set their bit;
//   exact   the queued (connection, box) pairs in ever finer parts and, those
//           still unsure, the exact trajectory-box test; a hit clears the bit;
//   degree  popcount of each row.
// A connection's bit ends set iff no box blocks it, the decision of the exact
// test on every box its range meets.
// ---------------------------------------------------------------------------
constexpr int kNearRows = 4;        // rows a workgroup takes together, one a wave in pass 2
constexpr int kNearThreads = 64 * kNearRows;
constexpr int kNearChunk = 1024;    // targets between two passes
constexpr int kNearKeep = 1536;     // pairs from which they are steered

__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Append `ok` items of a wave to a list: one atomic per wave (all 64 lanes
// call it).  Returns the slot of this lane's item.
__device__ __forceinline__ int wave_append(bool ok, int32_t* counter) {
    const unsigned long long m = __ballot(ok);
    const int lane = threadIdx.x & 63;
    int base = 0;
    if (lane == 0 && m) base = atomicAdd(counter, (int)__popcll(m));
    base = __shfl(base, 0, 64);
    return base + (int)__popcll(m & (lane ? ((1ull << lane) - 1ull) : 0ull));
}

__device__ __forceinline__ void gw_push_near(const GraphWork& gw, bool ok, int src, int dst,
                                             double tau) {
    const int slot = wave_append(ok, gw.counts + 0);
    if (ok && slot < gw.near_cap) {
        gw.near_src[slot] = src;
        gw.near_dst[slot] = dst;
        gw.near_tau[slot] = tau;
    }
}

// The same for a whole workgroup (all threads call it): one global atomic
// per workgroup and call, since every near connection of every row bumps the
// same counter.  s_w: [blockDim.x / 64 + 1] ints of LDS.
__device__ __forceinline__ void gw_push_near_block(const GraphWork& gw, bool ok, int src, int dst,
                                                   double tau, int* s_w) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const unsigned long long m = __ballot(ok);
    if (lane == 0) s_w[w] = (int)__popcll(m);
    __syncthreads();
    if (threadIdx.x == 0) {
        int tot = 0;
        for (int k = 0; k < nw; ++k) {
            const int c = s_w[k];
            s_w[k] = tot;
            tot += c;
        }
        s_w[nw] = tot ? atomicAdd(gw.counts + 0, tot) : 0;
    }
    __syncthreads();
    const int slot = s_w[nw] + s_w[w] + (int)__popcll(m & (lane ? ((1ull << lane) - 1ull) : 0ull));
    if (ok && slot < gw.near_cap) {
        gw.near_src[slot] = src;
        gw.near_dst[slot] = dst;
        gw.near_tau[slot] = tau;
    }
    __syncthreads();   // s_w is reused
}

// near: rows v0 .. v0 + rows - 1 (at most kNearRows) against targets u0 .. u1 - 1
// (whole workgroup).  Three passes, each over what the one before it leaves, so
// that no wave carries lanes the pass has no work for:
//   1. the first look at the Bernstein bound, a lane per target for all rows:
//      the target is loaded once, and its outcome is a bit of a ballot;
//   2. a wave per row, over the row's bits: the split bound;
//   3. the root solve (tau*, c*) over the pairs that keeps, of all rows, those
//      whose solve likely takes steer64's one-root branch from the front of the
//      list and the others from its end, each in waves of their own.
// It is bound by its instructions: of the 20,000-sample indoor query's pairs 18 %
// pass the first look and 5 % are steered, some 900 instructions each.  A row
// at a time, with FP64 for pass 2 and a list written from pass 1, it took 2.45
// ms; now 1.39 (64 uneven queries: 10.5 and 5.5).
struct NearLds {
    unsigned long long mask[kNearRows][kNearChunk / 64];
    uint16_t open[kNearRows][kNearChunk];                    // pass 1 -> 2
    uint32_t keep[kNearKeep + kNearRows * kNearChunk];       // pass 2 -> 3: row << 30 | target
    int n_one, n_many;
    int slots[kNearRows + 1];
};

__device__ __forceinline__ void near_steer(const float* __restrict__ X, int v0, double r_steer, double r_conn,
                                           const GraphWork& gw, NearLds& s) {
    constexpr int kCap = kNearKeep + kNearRows * kNearChunk;
    const int n_one = s.n_one, n_many = s.n_many;
    const int first_many = (n_one + 63) & ~63, end = first_many + n_many;
    for (int base = 0; base < end; base += kNearThreads) {
        const int i = base + threadIdx.x;
        const int at = i < n_one ? i : (i >= first_many && i < end ? kCap - 1 - (i - first_many) : -1);
        bool ok = false;
        int u = 0, v = 0;
        double tau = 0.0;
        if (at >= 0) {
            const uint32_t e = s.keep[at];
            u = (int)(e & 0x3fffffffu);
            v = v0 + (int)(e >> 30);
            double c;
            steer64(X + (size_t)v * 6, X + (size_t)u * 6, r_steer, tau, c);
            ok = c < r_conn && tau > kTauMin;
        }
        gw_push_near_block(gw, ok, v, u, tau, s.slots);
    }
}

__device__ __forceinline__ void gw_near_rows(const float* __restrict__ X,
                                             const uint8_t* __restrict__ valid, int v0, int rows, int u0,
                                             int u1, double r_steer, double r_conn, const GraphWork& gw,
                                             NearLds& s) {
    constexpr int kCap = kNearKeep + kNearRows * kNearChunk;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const Near32 k = near32((float)r_steer, (float)r_conn);
    float xv[kNearRows][6];
    bool on[kNearRows];
#pragma unroll
    for (int r = 0; r < kNearRows; ++r) {
        const int v = v0 + min(r, rows - 1);
        on[r] = r < rows && valid[v];
        for (int e = 0; e < 6; ++e) xv[r][e] = uniform(X[(size_t)v * 6 + e]);
    }
    const float* xw = X + (size_t)(v0 + min(wave, rows - 1)) * 6;   // this wave's row
    if (threadIdx.x == 0) s.n_one = s.n_many = 0;
    for (int c0 = u0; c0 < u1; c0 += kNearChunk) {
#pragma unroll 1
        for (int j = wave; j < kNearChunk / 64; j += kNearRows) {
            const int u = c0 + 64 * j + lane;
            const bool there = u < u1 && valid[min(u, u1 - 1)];
            const float2* xu2 = reinterpret_cast<const float2*>(X + (size_t)min(u, u1 - 1) * 6);
            const float2 p01 = xu2[0], p2v0 = xu2[1], v12 = xu2[2];
            const float xu[6] = {p01.x, p01.y, p2v0.x, p2v0.y, v12.x, v12.y};
#pragma unroll
            for (int r = 0; r < kNearRows; ++r) {
                float b[5], m;
                const bool open = !near_bern32(k, near_sums32(xv[r], xu), b, m);
                const unsigned long long bits = __ballot(open && there && u != v0 + r);
                if (lane == r) s.mask[r][j] = on[r] ? bits : 0ull;
            }
        }
        __syncthreads();
        // this wave's row: its open targets side by side, then their split bound
        int n_open = 0;
        {
            uint32_t bits = (uint32_t)(s.mask[wave][lane >> 2] >> (16 * (lane & 3))) & 0xffffu;
            const int mine = __popc(bits);
            int x = mine;
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(x, o, 64);
                if (lane >= o) x += y;
            }
            n_open = __shfl(x, 63, 64);
            int at = x - mine;
            while (bits) {
                s.open[wave][at++] = (uint16_t)(16 * lane + __ffs((int)bits) - 1);
                bits &= bits - 1u;
            }
            wave_lds_sync();
        }
        for (int i = lane; i < n_open; i += 64) {
            const int u = c0 + s.open[wave][i];
            const float2* xu2 = reinterpret_cast<const float2*>(X + (size_t)u * 6);
            const float2 p01 = xu2[0], p2v0 = xu2[1], v12 = xu2[2];
            const float xu[6] = {p01.x, p01.y, p2v0.x, p2v0.y, v12.x, v12.y};
            const Sums32 sm = near_sums32(xw, xu);
            float b[5], m;
            near_bern32(k, sm, b, m);
            if (!near_split32(b, m)) {
                const uint32_t e = (uint32_t)wave << 30 | (uint32_t)u;
                if (likely_one_root(sm, (float)r_steer))
                    s.keep[atomicAdd(&s.n_one, 1)] = e;
                else
                    s.keep[kCap - 1 - atomicAdd(&s.n_many, 1)] = e;
            }
        }
        __syncthreads();
        if (s.n_one + s.n_many > kNearKeep || c0 + kNearChunk >= u1) {
            near_steer(X, v0, r_steer, r_conn, gw, s);
            __syncthreads();
            if (threadIdx.x == 0) s.n_one = s.n_many = 0;
            __syncthreads();
        }
    }
}

// near for the column of node 0: thread p is the pair (p + 1) -> 0 (all
// lanes of a wave call it)
__device__ __forceinline__ void gw_near_col0(const float* __restrict__ X,
                                             const uint8_t* __restrict__ valid, int n, int p,
                                             double r_steer, double r_conn, const GraphWork& gw) {
    const int src = p + 1;
    bool ok = false;
    double tau = 0.0;
    if (src < n && valid[0] && valid[src] &&
        !surely_not_near(X + (size_t)src * 6, X, (float)r_steer, (float)r_conn)) {
        double c;
        steer64(X + (size_t)src * 6, X, r_steer, tau, c);
        ok = c < r_conn && tau > kTauMin;
    }
    gw_push_near(gw, ok, src, 0, tau);
}

// boxes over one list of connections (src, dst, tau, optional cached range).
// Exact-queue entries name the connection by `tag` (>= 0: index into the
// roadmap list, < 0: -1 - index into the near list).  check_valid: skip
// connections with an invalid end (the cached roadmap list).
//
// What bounds it is lanes without work: which boxes a connection comes near,
// and how far each must be looked into, differs from lane to lane.  So a wave
// takes 64 connections, lane by lane, only as far as every lane does the same
// -- the cubic, then its 8 pieces one after the other, each with the boxes that
// its extents' bins hold (FP32, in units of bins, widened by a bound of the
// rounding) -- and what differs goes through two
// queues in the wave's LDS, each worked on 64 entries at a time:
//   1. (connection, piece, box), the box met by the piece's extents in FP32:
//      the hull of the piece against the box in FP64.  It may miss the box (as
//      piece_clear), or prove a hit: it lies inside the box's slabs on two
//      axes, by kHullMargin, while its end values on the third enclose a value
//      inside that slab by the same margin (the third coordinate passes through
//      its slab while the other two stay in theirs; a thin wall crossed inside
//      its extent is settled this way);
//   2. those left: the piece's end and quarters; a sample point (not the
//      trajectory's own ends) inside the box proves a hit, and a box that some
//      quarter's hull still meets is left to the exact stage.
// A connection that a hit blocks drops out.  The indoor query of 20,000 samples
// (20.3 million connections, 6 in 10 blocked, 1.4 entries of queue 1 and 0.3 of
// queue 2 each) took 3.53 ms in this kernel with a lane per connection for all
// of it (29 % of the lanes with work) and a step of the exact list's counter for
// each connection's boxes; now it takes 1.38 (1.29 while its list came a row at a
// time from the near stage).
constexpr int kBoxThreads = 256;
constexpr int kBoxWaves = kBoxThreads / 64;
constexpr int kPieces = 8;
constexpr int kBoxQueue = 128;   // 63 left + 64 new

// One wave's LDS.
struct BoxWaveLds {
    double c23[6][64], tau[64];              // cubics: c2, c3 per axis
    float c01[6][64];                        // and c0, c1 (the start's FP32 state)
    uint32_t q1[kBoxQueue], q2[kBoxQueue];   // connection | piece << 6 | box << 9
    int x_edge[kBoxQueue], x_box[kBoxQueue]; // for the exact stage
    int blocked[64];
};

// Workgroup's dynamic LDS: per wave its BoxWaveLds, then per connection the
// boxes left to the exact stage, then the boxes and their bins.
__host__ __device__ inline size_t gw_boxes_lds(int n_obs) {
    return sizeof(BoxWaveLds) * kBoxWaves + (size_t)kBoxThreads * ((n_obs + 63) / 64) * 8 +
           (size_t)(bin_words(n_obs) - kBinHeader) * 4 + (size_t)n_obs * 48;
}

struct BoxStage {
    BoxWaveLds* w;               // this wave's
    uint32_t* left;              // [64][2 nw] bits of the boxes left to the exact stage
    const float* obs;
    const float* obs_bins;       // the boxes in units of bins
    BinView bins;
    int n1, n2, nx;              // queue lengths (wave-uniform)
};

__device__ __forceinline__ Cubic axis_cubic(const BoxWaveLds& l, int c, int a) {
    return Cubic{(double)l.c01[2 * a][c], (double)l.c01[2 * a + 1][c], l.c23[2 * a][c], l.c23[2 * a + 1][c]};
}

// Time of piece end k.
__device__ __forceinline__ double piece_end(double tau, int k) {
    constexpr double inv = 1.0 / (double)kPieces;
    return k == kPieces ? tau : tau * (inv * (double)k);
}

// The last (at most 16) entries of queue 2, a lane per quarter.
__device__ __forceinline__ void box_quarters(BoxStage& g) {
    const int lane = threadIdx.x & 63, j = lane & 3;
    wave_lds_sync();
    const int n = min(g.n2, 16);
    g.n2 -= n;
    if ((lane >> 2) < n) {
        const uint32_t e = g.w->q2[g.n2 + (lane >> 2)];
        const int c = e & 63, k = (e >> 6) & 7, o = e >> 9;
        if (!g.w->blocked[c]) {
            const double tau = g.w->tau[c];
            const float* box = g.obs + o * 6;
            constexpr double inv = 1.0 / (double)kPieces;
            const double h = inv * tau, q3 = 0.25 * (h * (1.0 / 3.0)), t0 = tau * (inv * (double)k);
            const double ta = j == 0 ? piece_end(tau, k) : t0 + 0.25 * (double)j * h;
            const double tb = j == 3 ? piece_end(tau, k + 1) : t0 + 0.25 * (double)(j + 1) * h;
            bool sep = false, inside = true;
#pragma unroll 1
            for (int a = 0; a < 3; ++a) {
                const Cubic q = axis_cubic(*g.w, c, a);
                const double pa = q.at(ta), pb = q.at(tb);
                const double b1 = pa + q3 * q.slope(ta), b2 = pb - q3 * q.slope(tb);
                const double lo = fmin(fmin(pa, pb), fmin(b1, b2)) - kHullMargin;
                const double hi = fmax(fmax(pa, pb), fmax(b1, b2)) + kHullMargin;
                const double blo = (double)box[a], bhi = (double)box[3 + a];
                sep |= (hi < blo) | (lo > bhi);
                inside &= (pb >= blo) & (pb <= bhi);
            }
            if (inside && (j < 3 || k + 1 < kPieces))
                g.w->blocked[c] = 1;
            else if (!sep)
                atomicOr(&g.left[c * 2 * g.bins.nw + (o >> 5)], 1u << (o & 31));
        }
    }
    wave_lds_sync();
}

// Lanes before this one for which ok holds (all lanes call it).
__device__ __forceinline__ int wave_rank(bool ok) {
    const unsigned long long m = __ballot(ok);
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Appends to a wave's queue (all lanes call it); at most 64 entries.
__device__ __forceinline__ void box_push(uint32_t* q, int& n, bool ok, uint32_t e) {
    const int at = n + wave_rank(ok);
    if (ok) q[at] = e;
    n += (int)__popcll(__ballot(ok));
}

// The last (at most 64) entries of queue 1.
__device__ __forceinline__ void box_hulls(BoxStage& g) {
    const int lane = threadIdx.x & 63;
    wave_lds_sync();
    const int n = min(g.n1, 64);
    g.n1 -= n;
    bool open = false;
    uint32_t e = 0;
    if (lane < n) {
        e = g.w->q1[g.n1 + lane];
        const int c = e & 63, k = (e >> 6) & 7, o = e >> 9;
        if (!g.w->blocked[c]) {
            const double tau = g.w->tau[c];
            const double h3 = (1.0 / (double)kPieces * tau) * (1.0 / 3.0);
            const double ta = piece_end(tau, k), tb = piece_end(tau, k + 1);
            const float* bx = g.obs + o * 6;
            bool sep = false;
            uint32_t in = 0, cr = 0;
#pragma unroll 1
            for (int a = 0; a < 3; ++a) {   // (an axis at a time: registers)
                const Cubic q = axis_cubic(*g.w, c, a);
                const double pa = q.at(ta), pb = q.at(tb);
                const double b1 = pa + h3 * q.slope(ta), b2 = pb - h3 * q.slope(tb);
                const double emin = fmin(pa, pb), emax = fmax(pa, pb);
                const double lo = fmin(emin, fmin(b1, b2)) - kHullMargin;
                const double hi = fmax(emax, fmax(b1, b2)) + kHullMargin;
                const double blo = (double)bx[a], bhi = (double)bx[3 + a];
                sep |= (hi < blo) | (lo > bhi);
                const double ilo = blo + kHullMargin, ihi = bhi - kHullMargin;
                in |= (uint32_t)((lo >= blo) & (hi <= bhi)) << a;
                cr |= (uint32_t)((ilo <= ihi) & (emin <= ihi) & (emax >= ilo)) << a;
            }
            const uint32_t out = 7u & ~in;   // axes on which it is not inside
            const bool hit = out == 0u ? cr != 0u : ((out & (out - 1u)) == 0u && (cr & out));
            if (!sep && hit) g.w->blocked[c] = 1;
            open = !sep && !hit;
        }
    }
    box_push(g.w->q2, g.n2, open, e);
    while (g.n2 >= 64) box_quarters(g);
    wave_lds_sync();
}

// The last (at most 64) entries for the exact stage to its list: one step of
// the list's counter, which all waves share, for all of them (with a step for
// every connection's boxes, 180,000 of them, the indoor query's stage took 2.28
// ms instead of 1.48).
__device__ __forceinline__ void box_exact_flush(BoxStage& g, const GraphWork& gw) {
    const int lane = threadIdx.x & 63;
    wave_lds_sync();
    const int n = min(g.nx, 64);
    g.nx -= n;
    int at = 0;
    if (lane == 0) at = atomicAdd(gw.counts + 1, n);
    at = __shfl(at, 0, 64) + lane;
    if (lane < n && at < gw.xq_cap) {
        gw.xq_edge[at] = g.w->x_edge[g.nx + lane];
        gw.xq_box[at] = g.w->x_box[g.nx + lane];
    }
    wave_lds_sync();
}

__device__ __forceinline__ bool boxes_apart(const float* lo, const float* hi, const float* bx) {
    return (hi[0] < bx[0]) | (lo[0] > bx[3]) | (hi[1] < bx[1]) | (lo[1] > bx[4]) | (hi[2] < bx[2]) |
           (lo[2] > bx[5]);
}

// Whole workgroup of kBoxThreads; lds: gw_boxes_lds(n_obs) bytes; bins: the
// query's table in memory (not read without boxes).
__device__ __forceinline__ void gw_boxes(const float* __restrict__ X,
                                         const uint8_t* __restrict__ valid,
                                         const int32_t* __restrict__ src_a,
                                         const int32_t* __restrict__ dst_a,
                                         const double* __restrict__ tau_a,
                                         const double* __restrict__ bbox, int count, bool near_list,
                                         bool check_valid, const float* __restrict__ obs, int n_obs,
                                         const uint32_t* __restrict__ bins, const GraphWork& gw,
                                         uint32_t* __restrict__ ebits, int words, int gid, int stride,
                                         char* lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    BoxStage g;
    g.w = reinterpret_cast<BoxWaveLds*>(lds) + wave;
    g.n1 = g.n2 = g.nx = 0;
    {
        const int nw = (n_obs + 63) / 64, n_set = bin_words(n_obs) - kBinHeader;
        uint32_t* left = reinterpret_cast<uint32_t*>(lds + sizeof(BoxWaveLds) * kBoxWaves);
        uint32_t* set = left + kBoxThreads * nw * 2;
        float* s_obs = reinterpret_cast<float*>(set + n_set);
        for (int t = threadIdx.x; t < n_set; t += kBoxThreads) set[t] = bins[kBinHeader + t];
        float* s_obs_bins = s_obs + n_obs * 6;
        for (int t = threadIdx.x; t < n_obs * 6; t += kBoxThreads) {
            const int a = t % 3;
            s_obs[t] = obs[t];
            s_obs_bins[t] = (obs[t] - __uint_as_float(bins[a])) * __uint_as_float(bins[3 + a]);
        }
        g.obs_bins = s_obs_bins;
        for (int a = 0; a < 3; ++a) {
            g.bins.org[a] = n_obs ? __uint_as_float(bins[a]) : 0.0f;
            g.bins.scale[a] = n_obs ? __uint_as_float(bins[3 + a]) : 0.0f;
        }
        g.bins.nw = nw;
        g.bins.set = reinterpret_cast<const unsigned long long*>(set);
        g.left = left + wave * 64 * nw * 2;
        g.obs = s_obs;
        for (int k = 0; k < 2 * nw; ++k) g.left[lane * 2 * nw + k] = 0u;
        __syncthreads();
    }
    const int nw = g.bins.nw;
    // all lanes of a wave iterate together (stride is a multiple of 64)
    for (int base = gid - lane; base < count; base += stride) {
        const int i = base + lane;
        bool keep = i < count;
        if (keep) keep = !check_valid || (valid[src_a[i]] && valid[dst_a[i]]);
        bool look = keep;
        if (bbox && look) {
            // a cached range that meets no box settles the connection
            float lo[3], hi[3];
            for (int a = 0; a < 3; ++a) {
                lo[a] = __double2float_rd(bbox[(size_t)i * 6 + a]);
                hi[a] = __double2float_ru(bbox[(size_t)i * 6 + 3 + a]);
            }
            BinRange r;
            bin_range(g.bins, lo, hi, r);
            look = false;
            for (int w = 0; w < nw && !look; ++w) look = bin_candidates(g.bins, r, w) != 0ull;
        }
        g.w->blocked[lane] = 0;
        if (__ballot(look) != 0ull) {
            // q(u) = (p - org) * scale, u = piece units: k0 + u (k1 + u (k2 + u k3))
            float k0[3], k1[3], k2[3], k3[3], pad[3];
            for (int a = 0; a < 3; ++a) k0[a] = k1[a] = k2[a] = k3[a] = pad[a] = 0.0f;
            if (look) {
                Cubic cs[3];
                const double tau = tau_a[i], h = tau * (1.0 / (double)kPieces);
                hermite(X + (size_t)src_a[i] * 6, X + (size_t)dst_a[i] * 6, tau, cs);
                g.w->tau[lane] = tau;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    g.w->c01[2 * a][lane] = (float)cs[a].c0;
                    g.w->c01[2 * a + 1][lane] = (float)cs[a].c1;
                    g.w->c23[2 * a][lane] = cs[a].c2;
                    g.w->c23[2 * a + 1][lane] = cs[a].c3;
                    const double sc = (double)g.bins.scale[a], org = (double)g.bins.org[a];
                    k0[a] = (float)((cs[a].c0 - org) * sc);
                    k1[a] = (float)(cs[a].c1 * (sc * h));
                    k2[a] = (float)(cs[a].c2 * (sc * h * h));
                    k3[a] = (float)(cs[a].c3 * (sc * h * h * h));
                    // The coefficients, the Horner steps of the piece ends and the
                    // control points round at most some 12 times by 2^-24 of
                    // sums no larger than this; a box's ends three times by
                    // 2^-24 of themselves and of 16 * scale (|org| at most 16).
                    const float mag = fabsf(k0[a]) + 8.0f * fabsf(k1[a]) + 64.0f * fabsf(k2[a]) + 512.0f * fabsf(k3[a]);
                    pad[a] = 0x1p-18f * (mag + (float)kBins + 16.0f * g.bins.scale[a]) +
                             2.0f * (float)kHullMargin * g.bins.scale[a];
                    if (!(mag <= 1e30f)) {   // (no bound: every box)
                        k0[a] = k1[a] = k2[a] = k3[a] = 0.0f;
                        pad[a] = INFINITY;
                    }
                }
            }
            float qa[3], ea[3];   // a piece's start, and a third of its length along the tangent
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                qa[a] = k0[a];
                ea[a] = k1[a] * (1.0f / 3.0f);
            }
#pragma unroll 1
            for (int k = 0; k < kPieces; ++k) {
                const float u = (float)(k + 1);
                float lo[3], hi[3];
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const float qb = k0[a] + u * (k1[a] + u * (k2[a] + u * k3[a]));
                    const float eb = (k1[a] + u * (2.0f * k2[a] + u * (3.0f * k3[a]))) * (1.0f / 3.0f);
                    const float c1 = qa[a] + ea[a], c2 = qb - eb;
                    lo[a] = fminf(fminf(qa[a], qb), fminf(c1, c2)) - pad[a];
                    hi[a] = fmaxf(fmaxf(qa[a], qb), fmaxf(c1, c2)) + pad[a];
                    qa[a] = qb;
                    ea[a] = eb;
                }
                look = look && !g.w->blocked[lane];
                if (__ballot(look) == 0ull) break;
                for (int w = 0; w < nw; ++w) {
                    unsigned long long m = 0ull;
                    if (look) {
                        BinRange r;
#pragma unroll
                        for (int a = 0; a < 3; ++a) {
                            const int bh = (int)fminf(fmaxf(hi[a], 0.0f), (float)(kBins - 1));
                            const int bl = (int)fminf(fmaxf(lo[a], 0.0f), (float)(kBins - 1));
                            r.le[a] = (a * kBins + bh) * nw;
                            r.ge[a] = (3 * kBins + a * kBins + bl) * nw;
                        }
                        m = bin_candidates(g.bins, r, w);
                    }
                    while (__ballot(m != 0ull) != 0ull) {
                        const int o = w * 64 + (m ? __ffsll((long long)m) - 1 : 0);
                        const bool met = m && !boxes_apart(lo, hi, g.obs_bins + o * 6);
                        m &= m - 1ull;
                        box_push(g.w->q1, g.n1, met, (uint32_t)lane | (uint32_t)k << 6 | (uint32_t)o << 9);
                        if (g.n1 >= 64) box_hulls(g);
                    }
                }
            }
            while (g.n1) box_hulls(g);
            while (g.n2) box_quarters(g);
            // what the quarters left open, if the connection's range meets the box
            wave_lds_sync();
            for (int w = 0; w < 2 * nw; ++w) {
                uint32_t m = g.left[lane * 2 * nw + w];
                if (m) g.left[lane * 2 * nw + w] = 0u;
                if (g.w->blocked[lane]) m = 0u;
                float lo[3] = {0.f, 0.f, 0.f}, hi[3] = {0.f, 0.f, 0.f};
                if (m) {
                    for (int a = 0; a < 3; ++a) {
                        double mn, mx;
                        if (bbox) {
                            mn = bbox[(size_t)i * 6 + a];
                            mx = bbox[(size_t)i * 6 + 3 + a];
                        } else {
                            cubic_range(axis_cubic(*g.w, lane, a), g.w->tau[lane], mn, mx);
                        }
                        lo[a] = __double2float_rd(mn);
                        hi[a] = __double2float_ru(mx);
                    }
                }
                while (__ballot(m != 0u) != 0ull) {
                    const int o = w * 32 + (m ? __ffs((int)m) - 1 : 0);
                    const bool ask = m && !boxes_apart(lo, hi, g.obs + o * 6);
                    m &= m - 1u;
                    const int at = g.nx + wave_rank(ask);
                    if (ask) {
                        g.w->x_edge[at] = near_list ? -1 - i : i;
                        g.w->x_box[at] = o;
                    }
                    g.nx += (int)__popcll(__ballot(ask));
                    if (g.nx >= 64) box_exact_flush(g, gw);
                }
            }
        }
        if (keep && !g.w->blocked[lane]) {
            const int dst = dst_a[i];
            atomicOr(&ebits[(size_t)src_a[i] * words + (dst >> 5)], 1u << (dst & 31));
        }
        wave_lds_sync();
    }
    if (g.nx) box_exact_flush(g, gw);
}

// exact: queued (connection, box) pairs; a hit clears the connection's bit.
// A wave takes up to 64 pairs and refines them over its lanes: the 8 pieces of 8
// pairs at a time; 8 parts of each piece that met the box (through a queue), and
// 4 of each part; a sample point inside the box proves a hit.  Pairs that stay
// open -- a graze, mostly -- are solved for the slab crossings, a lane for each
// axis and monotone piece.  With a wave per pair, its 64 parts on the lanes and
// the crossings solved by all lanes alike, the 20,000-sample indoor query took
// 0.40 ms here, 64 uneven queries 1.64; now 0.12 and 0.36.
struct ExactWaveLds {
    double c23[6][64], tau[64];
    float c01[6][64], box[6][64];
    uint16_t q1[kBoxQueue], q2[kBoxQueue];   // pair | part << 6
    int state[64];                           // 1 hit, 2 open
    int solve[kBoxQueue];                    // pairs for the crossings
};

// Part idx of `parts` of pair c: 0 clear, 1 hit, 2 open.
__device__ __forceinline__ int exact_part(const ExactWaveLds& l, int c, int idx, int parts) {
    const double tau = l.tau[c], inv = 1.0 / (double)parts;
    const double h3 = (inv * tau) * (1.0 / 3.0);
    const double ta = tau * (inv * (double)idx);
    const double tb = idx + 1 == parts ? tau : tau * (inv * (double)(idx + 1));
    bool sep = false, inside = idx + 1 < parts;
#pragma unroll 1
    for (int a = 0; a < 3; ++a) {
        const Cubic q{(double)l.c01[2 * a][c], (double)l.c01[2 * a + 1][c], l.c23[2 * a][c], l.c23[2 * a + 1][c]};
        const double pa = q.at(ta), pb = q.at(tb);
        const double b1 = pa + h3 * q.slope(ta), b2 = pb - h3 * q.slope(tb);
        const double lo = fmin(fmin(pa, pb), fmin(b1, b2)) - kHullMargin;
        const double hi = fmax(fmax(pa, pb), fmax(b1, b2)) + kHullMargin;
        const double blo = (double)l.box[a][c], bhi = (double)l.box[3 + a][c];
        sep |= (hi < blo) | (lo > bhi);
        inside &= (pb >= blo) & (pb <= bhi);
    }
    return inside ? 1 : (sep ? 0 : 2);
}

__device__ __forceinline__ void gw_exact(const float* __restrict__ X, const float* __restrict__ obs,
                                         const GraphWork& gw, const int32_t* __restrict__ rm_src,
                                         const int32_t* __restrict__ rm_dst,
                                         const double* __restrict__ rm_tau,
                                         uint32_t* __restrict__ ebits, int words, int gid,
                                         int stride, ExactWaveLds* lds) {
    const int lane = threadIdx.x & 63;
    ExactWaveLds& l = lds[threadIdx.x >> 6];
    const int N = min(gw.counts[1], gw.xq_cap);
    // pairs a wave: 64 where there are enough of them, else enough waves
    const int waves = stride >> 6;
    const int group = min(64, ((N + waves - 1) / waves + 7) & ~7);
    auto ends = [&](int i, int& src, int& dst, double& tau) {
        const int tag = gw.xq_edge[i];
        if (tag >= 0) {
            src = rm_src[tag]; dst = rm_dst[tag]; tau = rm_tau[tag];
        } else {
            src = gw.near_src[-1 - tag]; dst = gw.near_dst[-1 - tag]; tau = gw.near_tau[-1 - tag];
        }
    };
    auto clear = [&](int src, int dst) {
        atomicAnd(&ebits[(size_t)src * words + (dst >> 5)], ~(1u << (dst & 31)));
    };
    int n_solve = 0;
    // the last (at most 4), 16 lanes each: lane 3 a + k of a pair finds the time
    // in the slab of axis a on its monotone piece k; three of them, one an axis,
    // that share a time are a hit
    auto solve = [&]() {
        wave_lds_sync();
        const int n = min(n_solve, 4), who = lane >> 4, sub = lane & 15, first = lane & 48;
        n_solve -= n;
        double in = INFINITY, out = -INFINITY;
        int src = 0, dst = 0;
        if (who < n && sub < 9) {
            const int i = l.solve[n_solve + who];
            double tau;
            ends(i, src, dst, tau);
            const int a = sub / 3;
            const float* x0 = X + (size_t)src * 6 + a;
            const float* x1 = X + (size_t)dst * 6 + a;
            const float* bx = obs + (size_t)gw.xq_box[i] * 6 + a;
            const Cubic c = hermite_axis(x0[0], x0[3], x1[0], x1[3], tau, 1.0 / tau);
            slab_piece(c, tau, (double)bx[0], (double)bx[3], sub - 3 * a, in, out);
        }
        const int ja = first + sub / 3, jb = first + 3 + sub % 3;
        const double st = fmax(__shfl(in, ja, 64), __shfl(in, jb, 64));
        const double en = fmin(__shfl(out, ja, 64), __shfl(out, jb, 64));
        bool hit = false;
        for (int k = 0; k < 3; ++k) {
            const double s2 = __shfl(in, first + 6 + k, 64), e2 = __shfl(out, first + 6 + k, 64);
            hit |= fmax(st, s2) <= fmin(en, e2);
        }
        const unsigned long long hits = __ballot(hit && sub < 9) >> first & 0xffffull;
        if (who < n && sub == 0 && hits) clear(src, dst);
        wave_lds_sync();
    };
    for (int base = (gid >> 6) * group; base < N; base += waves * group) {
        const int n = min(group, N - base);
        const bool last = base + waves * group >= N;
        int src = 0, dst = 0;
        if (lane < n) {
            double tau;
            ends(base + lane, src, dst, tau);
            Cubic cs[3];
            hermite(X + (size_t)src * 6, X + (size_t)dst * 6, tau, cs);
            const float* bx = obs + (size_t)gw.xq_box[base + lane] * 6;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                l.c01[2 * a][lane] = (float)cs[a].c0;
                l.c01[2 * a + 1][lane] = (float)cs[a].c1;
                l.c23[2 * a][lane] = cs[a].c2;
                l.c23[2 * a + 1][lane] = cs[a].c3;
                l.box[a][lane] = bx[a];
                l.box[3 + a][lane] = bx[3 + a];
            }
            l.tau[lane] = tau;
            l.state[lane] = 0;
        }
        wave_lds_sync();
        int n1 = 0, n2 = 0;
        auto quarters = [&]() {   // the last (at most 16) of q2, 4 lanes each
            wave_lds_sync();
            const int m = min(n2, 16);
            n2 -= m;
            if ((lane >> 2) < m) {
                const int e = l.q2[n2 + (lane >> 2)], c = e & 63;
                if (l.state[c] != 1) {
                    const int r = exact_part(l, c, 4 * (e >> 6) + (lane & 3), 256);
                    if (r == 1) atomicExch(&l.state[c], 1);
                    if (r == 2) atomicCAS(&l.state[c], 0, 2);
                }
            }
            wave_lds_sync();
        };
        auto eighths = [&]() {    // the last (at most 8) of q1, 8 lanes each
            wave_lds_sync();
            const int m = min(n1, 8);
            n1 -= m;
            bool open = false;
            int c = 0, idx = 0;
            if ((lane >> 3) < m) {
                const int e = l.q1[n1 + (lane >> 3)];
                c = e & 63;
                idx = 8 * (e >> 6) + (lane & 7);
                if (l.state[c] != 1) {
                    const int r = exact_part(l, c, idx, 64);
                    if (r == 1) l.state[c] = 1;
                    open = r == 2;
                }
            }
            const int at = n2 + wave_rank(open);
            if (open) l.q2[at] = (uint16_t)(c | idx << 6);
            n2 += (int)__popcll(__ballot(open));
            while (n2 >= 64) quarters();
            wave_lds_sync();
        };
        for (int b0 = 0; b0 < n; b0 += 8) {
            const int c = b0 + (lane >> 3), idx = lane & 7;
            bool open = false;
            if (c < n) {
                const int r = exact_part(l, c, idx, 8);
                if (r == 1) l.state[c] = 1;
                open = r == 2;
            }
            const int at = n1 + wave_rank(open);
            if (open) l.q1[at] = (uint16_t)(c | idx << 6);
            n1 += (int)__popcll(__ballot(open));
            while (n1 >= 64) eighths();
        }
        while (n1 > 0) eighths();
        while (n2 > 0) quarters();
        wave_lds_sync();
        const int st = lane < n ? l.state[lane] : 0;
        if (st == 1) clear(src, dst);
        const int at = n_solve + wave_rank(st == 2);
        if (st == 2) l.solve[at] = base + lane;
        n_solve += (int)__popcll(__ballot(st == 2));
        while (n_solve >= (last ? 1 : 4)) solve();
        wave_lds_sync();
    }
}

// degree: out-degree of each row of the bit matrix (one wave per row)
__device__ __forceinline__ void row_deg_dev(const uint32_t* __restrict__ ebits, int n_nodes, int words,
                                            int32_t* __restrict__ deg, int v) {
    const int lane = threadIdx.x & 63;
    if (v >= n_nodes) return;
    int d = 0;
    for (int w = lane; w < words; w += 64) d += __popc(ebits[(size_t)v * words + w]);
    for (int o = 32; o > 0; o >>= 1) d += __shfl_down(d, o, 64);
    if (lane == 0) deg[v] = d;
}

__device__ __forceinline__ void graph_fill_dev(int n, const uint32_t* __restrict__ ebits,
                                                    const int32_t* __restrict__ row_ptr,
                                                    int32_t* __restrict__ col,
                                                    int32_t* __restrict__ esrc, int words) {
    // one wave per row, one 32-bit word of the row per lane and pass: the
    // lanes' bit counts scanned across the wave give each lane its first
    // slot, and the lane writes its word's columns in ascending order
    const int v = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (v >= n) return;
    int pos = row_ptr[v];
    for (int w0 = 0; w0 < words; w0 += 64) {
        const int w = w0 + lane;
        uint32_t bits = w < words ? ebits[(size_t)v * words + w] : 0u;
        const int c = __popc(bits);
        int x = c;
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        int at = pos + x - c;
        while (bits) {
            const int b = __ffs((int)bits) - 1;
            bits &= bits - 1u;
            col[at] = w * 32 + b;
            esrc[at] = v;
            ++at;
        }
        pos += __shfl(x, 63, 64);
    }
}

// Pass 2 from the near list, without steering again.  The near list holds
// each connection's tau* from pass 1 and every graph edge is one of its
// entries whose bit survived the box and exact stages, so:
//   word_start_dev: the CSR slot of the first edge of each 32-bit word of
//     each row (one wave per row, the words' bit counts scanned);
//   near_to_slot_dev: each surviving near entry's slot (its word's start
//     plus the bits below it in the word) receives its tau* -- in ecost,
//     since etau still holds the near list;
//   edge_cost_dev (after graph_fill_dev): tau* to etau and c* = cost_of(tau*)
//     to ecost, the very expression steer64 returns, so (tau*, c*) equal
//     what a second steering would give, bit for bit.
__device__ __forceinline__ void word_start_dev(int n, const uint32_t* __restrict__ ebits,
                                               const int32_t* __restrict__ row_ptr,
                                               int32_t* __restrict__ wstart, int words) {
    const int v = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (v >= n) return;
    int pos = row_ptr[v];
    for (int w0 = 0; w0 < words; w0 += 64) {
        const int w = w0 + lane;
        const int c = w < words ? __popc(ebits[(size_t)v * words + w]) : 0;
        int x = c;
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (w < words) wstart[(size_t)v * words + w] = pos + x - c;
        pos += __shfl(x, 63, 64);
    }
}

__device__ __forceinline__ void near_to_slot_dev(const GraphWork& gw, const uint32_t* __restrict__ ebits,
                                                 const int32_t* __restrict__ wstart, int words,
                                                 double* __restrict__ slot_tau) {
    const int count = min(gw.counts[0], gw.near_cap);
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) {
        const int v = gw.near_src[i], u = gw.near_dst[i];
        const size_t wi = (size_t)v * words + (u >> 5);
        const uint32_t word = ebits[wi];
        const uint32_t bit = 1u << (u & 31);
        if (word & bit) slot_tau[wstart[wi] + __popc(word & (bit - 1u))] = gw.near_tau[i];
    }
}

__device__ __forceinline__ void edge_cost_dev(const float* __restrict__ X, int n, double r_steer,
                                              const int32_t* __restrict__ row_ptr,
                                              const int32_t* __restrict__ col,
                                              const int32_t* __restrict__ esrc,
                                              double* __restrict__ etau, double* __restrict__ ecost) {
    const int E = row_ptr[n];
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < E; e += gridDim.x * blockDim.x) {
        const double tau = ecost[e];
        const BSums s = boundary_sums(X + (size_t)esrc[e] * 6, X + (size_t)col[e] * 6);
        etau[e] = tau;
        ecost[e] = cost_of(tau, s, r_steer);
    }
}

// Edge controls, one lane per edge: the same FP64 steering as pass 1, so the
// cached (tau*, c*) are bit-identical to the values that admitted the edge.
__device__ __forceinline__ void edge_steer_dev(const float* __restrict__ X, int n,
                                                    double r_steer,
                                                    const int32_t* __restrict__ row_ptr,
                                                    const int32_t* __restrict__ col,
                                                    const int32_t* __restrict__ esrc,
                                                    double* __restrict__ etau,
                                                    double* __restrict__ ecost) {
    const int E = row_ptr[n];
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < E; e += gridDim.x * blockDim.x) {
        const float* xv = X + (size_t)esrc[e] * 6;
        const float* xu = X + (size_t)col[e] * 6;
        double tau, c;
        steer64(xv, xu, r_steer, tau, c);
        etau[e] = tau;
        ecost[e] = c;
    }
}


}  // namespace pump
