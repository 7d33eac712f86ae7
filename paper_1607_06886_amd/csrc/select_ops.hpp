// Per-query operations of PlanSelection (Alg. 5), shared by the single-query
// kernels and the batched engine.
#pragma once

#include "device_math.hpp"
#include "pump_internal.hpp"

namespace pump {

// P_goal = plans still in P(v) for goal nodes v (Alg. 4 return), in id order
// (whole block; blockDim.x a multiple of 64, at most 1024).  a.n_plans < 0:
// the plan count is read from the control block (Explore still in flight on
// the stream when the host enqueued this).
__device__ __forceinline__ void goal_collect_block(const SelectArgs& a) {
    const int n_plans = a.n_plans >= 0 ? a.n_plans : a.ctl->n_plans;
    __shared__ int s_w[16];
    __shared__ int s_base;
    const int nw = blockDim.x >> 6;
    if (threadIdx.x == 0) s_base = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int b0 = 0; b0 < n_plans; b0 += blockDim.x) {
        const int p = b0 + threadIdx.x;
        const bool f = p < n_plans && a.p_state[p] != kRemoved && a.goal[a.p_head[p]];
        const unsigned long long m = __ballot(f);
        if (lane == 0) s_w[wave] = __popcll(m);
        __syncthreads();
        int off = s_base;
        for (int w = 0; w < wave; ++w) off += s_w[w];
        const int pos = off + (int)__popcll(m & (lane ? ((1ull << lane) - 1ull) : 0ull));
        if (f && pos < kMaxGoal) a.goal_ids[pos] = p;
        __syncthreads();
        if (threadIdx.x == 0) {
            int t = 0;
            for (int w = 0; w < nw; ++w) t += s_w[w];
            s_base += t;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) a.ctl->n_goal = s_base;
}

// Pareto front of P_goal (d dominates p iff p.cost > d.cost and
// p.pop >= d.pop), sorted by pop ascending, cost descending, then node
// sequence.  Paths are reconstructed from the parent links.
__device__ __forceinline__ int path_of(const SelectArgs& a, int p, int* out, int cap) {
    int n = 0;
    for (int q = p; q >= 0 && n < cap; q = a.p_parent[q]) out[n++] = a.p_head[q];
    for (int i = 0; i < n / 2; ++i) { int t = out[i]; out[i] = out[n - 1 - i]; out[n - 1 - i] = t; }
    return n;
}

__device__ __forceinline__ bool front_less(const SelectArgs& a, int fa, int fb) {
    const int pa = a.front_ids[fa], pb = a.front_ids[fb];
    if (a.p_pop[pa] != a.p_pop[pb]) return a.p_pop[pa] < a.p_pop[pb];
    if (a.p_cost[pa] != a.p_cost[pb]) return a.p_cost[pa] > a.p_cost[pb];
    const int stride = a.S_max + 1;
    const int* xa = a.paths + (size_t)fa * stride;
    const int* xb = a.paths + (size_t)fb * stride;
    const int la = a.path_len[fa], lb = a.path_len[fb];
    for (int i = 0; i < la && i < lb; ++i)
        if (xa[i] != xb[i]) return xa[i] < xb[i];
    return la < lb;
}

// Whole block; `max_front` bounds the front kept (kMaxFront or less).
// The dominance test takes the goal plans' (cost, pop) in LDS tiles; the
// front's paths are rebuilt by a thread each, ordered by one thread on an
// index array, and rebuilt once more in that order (no path is moved).
constexpr int kFrontTile = 256;

__device__ __forceinline__ void front_block(const SelectArgs& a, int max_front) {
    __shared__ int s_flag[kMaxFront];
    __shared__ int s_ord[kMaxFront];
    __shared__ double s_c[kFrontTile];
    __shared__ int s_k[kFrontTile];
    __shared__ int s_n;
    const int G = a.ctl->n_goal < kMaxGoal ? a.ctl->n_goal : kMaxGoal;
    if (threadIdx.x == 0) s_n = 0;
    for (int g0 = 0; g0 < G; g0 += blockDim.x) {   // (the same trip count in every thread)
        const int g = g0 + threadIdx.x;
        const bool have = g < G;
        double c = 0.0;
        int k = 0;
        if (have) {
            const int p = a.goal_ids[g];
            c = a.p_cost[p];
            k = a.p_pop[p];
        }
        bool dom = false;
        for (int h0 = 0; h0 < G; h0 += kFrontTile) {
            __syncthreads();
            for (int t = threadIdx.x; t < kFrontTile && h0 + t < G; t += blockDim.x) {
                const int d = a.goal_ids[h0 + t];
                s_c[t] = a.p_cost[d];
                s_k[t] = a.p_pop[d];
            }
            __syncthreads();
            const int hn = min(kFrontTile, G - h0);
            if (have)
                for (int h = 0; h < hn && !dom; ++h) dom = (c > s_c[h]) && (k >= s_k[h]);
        }
        if (have && !dom) {
            const int slot = atomicAdd(&s_n, 1);
            if (slot < max_front) s_flag[slot] = g;
        }
    }
    __syncthreads();
    const int n = s_n < max_front ? s_n : max_front;
    if (threadIdx.x == 0) {
        if (s_n > max_front) a.ctl->err = 2;
        // deterministic order of discovery: sort slots by goal index
        for (int i = 1; i < n; ++i) {
            const int v = s_flag[i];
            int j = i - 1;
            while (j >= 0 && s_flag[j] > v) { s_flag[j + 1] = s_flag[j]; --j; }
            s_flag[j + 1] = v;
        }
    }
    __syncthreads();
    const int stride = a.S_max + 1;
    for (int f = threadIdx.x; f < n; f += blockDim.x) {
        a.front_ids[f] = a.goal_ids[s_flag[f]];
        a.path_len[f] = path_of(a, a.front_ids[f], a.paths + (size_t)f * stride, stride);
        s_ord[f] = f;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        // insertion sort of the front's indices (pop, then cost, then path)
        for (int i = 1; i < n; ++i) {
            const int v = s_ord[i];
            int j = i - 1;
            while (j >= 0 && front_less(a, v, s_ord[j])) { s_ord[j + 1] = s_ord[j]; --j; }
            s_ord[j + 1] = v;
        }
    }
    __syncthreads();
    int id[(kMaxFront + 63) / 64];   // this thread's entries in the sorted order
    for (int f = threadIdx.x, r = 0; f < n; f += blockDim.x, ++r) id[r] = a.front_ids[s_ord[f]];
    __syncthreads();
    for (int f = threadIdx.x, r = 0; f < n; f += blockDim.x, ++r) {
        a.front_ids[f] = id[r];
        a.path_len[f] = path_of(a, id[r], a.paths + (size_t)f * stride, stride);
    }
    if (threadIdx.x == 0) a.ctl->n_front = n;
}

// Nominal tracking waypoints of path f (step 0 = the first node's position):
// each connection (u, v) contributes K_e = max(1, ceil(tau*/dt)) waypoints at
// t_k = k tau*/K_e.
__device__ __forceinline__ void waypoints_one(const SelectArgs& a, int f) {
    const int stride = a.S_max + 1;
    const int* nodes = a.paths + (size_t)f * stride;
    const int len = a.path_len[f];
    double* wp = a.wp + (size_t)f * stride * 3;
    const float* x0 = a.X + (size_t)nodes[0] * 6;
    for (int ax = 0; ax < 3; ++ax) wp[ax] = (double)x0[ax];
    int s = 0;
    bool ok = true;
    for (int l = 1; l < len && ok; ++l) {
        const float* xu = a.X + (size_t)nodes[l - 1] * 6;
        const float* xv = a.X + (size_t)nodes[l] * 6;
        double tau, c;
        steer64(xu, xv, a.r_steer, tau, c);
        const int K = max(1, (int)ceil(tau / a.dt));
        if (s + K > a.S_max) { ok = false; break; }
        Cubic cs[3];
        hermite(xu, xv, tau, cs);
        for (int k = 1; k <= K; ++k) {
            const double t = ((double)k * tau) / (double)K;
            for (int ax = 0; ax < 3; ++ax) wp[(size_t)(s + k) * 3 + ax] = cs[ax].at(t);
        }
        s += K;
    }
    a.wp_len[f] = ok ? s : -1;
}

// The same for one path by a whole wave (all 64 lanes call it): lane l takes
// the path's edges l + 1, l + 65, ...; the edges' waypoint counts are scanned
// across the wave for their offsets, so the root solves run side by side.
// Every waypoint is computed as in waypoints_one (same steer, same cubic,
// same t_k), so the table is identical; a path past S_max gets wp_len -1.
__device__ __forceinline__ void waypoints_wave(const SelectArgs& a, int f) {
    const int lane = threadIdx.x & 63;
    const int stride = a.S_max + 1;
    const int* nodes = a.paths + (size_t)f * stride;
    const int len = a.path_len[f];
    double* wp = a.wp + (size_t)f * stride * 3;
    if (lane == 0) {
        const float* x0 = a.X + (size_t)nodes[0] * 6;
        for (int ax = 0; ax < 3; ++ax) wp[ax] = (double)x0[ax];
    }
    int s0 = 0;                            // waypoints before this chunk of edges
    for (int l0 = 1; l0 < len; l0 += 64) {
        const int l = l0 + lane;
        double tau = 0.0;
        int K = 0;
        if (l < len) {
            double c;
            steer64(a.X + (size_t)nodes[l - 1] * 6, a.X + (size_t)nodes[l] * 6, a.r_steer, tau, c);
            K = max(1, (int)ceil(tau / a.dt));
        }
        int x = K;                         // inclusive scan of K over the lanes
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        const int s = s0 + x - K;          // this edge's first step - 1
        if (l < len) {
            Cubic cs[3];
            hermite(a.X + (size_t)nodes[l - 1] * 6, a.X + (size_t)nodes[l] * 6, tau, cs);
            for (int k = 1; k <= K && s + k <= a.S_max; ++k) {
                const double t = ((double)k * tau) / (double)K;
                for (int ax = 0; ax < 3; ++ax) wp[(size_t)(s + k) * 3 + ax] = cs[ax].at(t);
            }
        }
        s0 += __shfl(x, 63, 64);
    }
    if (lane == 0) a.wp_len[f] = s0 <= a.S_max ? s0 : -1;
}

// Alg. 5's choice among the risk-sorted front (cp_hat ascending): a
// bisection for the riskiest plan whose certification count stays within
// alpha, premised on MC growing along that order.  `good` (1-based) is the
// plan the search stands on -- it starts on the safest plan, not yet
// evaluated -- and plans from `bad` on are ruled out.  Each probe takes the
// middle of the open range: a count within alpha moves `good` up to it, one
// above alpha moves `bad` down to it.  Once nothing lies strictly between the
// two, `good` is checked once more (it may never have been probed).  Returns
// its 0-based index, or -1 when that check fails (infeasible) or nf < 1.
__device__ __forceinline__ int certified_pick(const int* mc_counts, int nf, int M, double alpha) {
    if (nf < 1) return -1;
    auto within = [&](int k) { return (double)mc_counts[k - 1] / (double)M <= alpha; };
    int good = 1, bad = nf + 1;
    while (bad - good > 1) {
        const int mid = (good + bad) >> 1;
        if (within(mid)) good = mid; else bad = mid;
    }
    return within(good) ? good - 1 : -1;
}

// Does the segment prev -> cur meet the closed box b?  Slab clipping in FP64
// after a bounding-box reject.
__device__ __forceinline__ bool segment_hits_box(const double prev[3], const double cur[3], const float* b) {
    bool apart = false;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax)
        apart |= (fmax(prev[ax], cur[ax]) < (double)b[ax]) | (fmin(prev[ax], cur[ax]) > (double)b[3 + ax]);
    if (apart) return false;   // a segment whose bounding box misses the box misses the box
    double t0 = 0.0, t1 = 1.0;
    bool miss = false;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const double d = cur[ax] - prev[ax];
        const double lo = (double)b[ax], hi = (double)b[3 + ax];
        if (d == 0.0) {
            miss |= (prev[ax] < lo) | (prev[ax] > hi);
        } else {
            const double ta = (lo - prev[ax]) / d, tb = (hi - prev[ax]) / d;
            t0 = fmax(t0, fmin(ta, tb));
            t1 = fmin(t1, fmax(ta, tb));
        }
    }
    return !miss && t0 <= t1;
}

// ---------------------------------------------------------------------------
// MC(p): certification particle m follows the closed-loop recurrence from zero
// with its own noise (under LQG tracking the joint state (dp, dv, p_hat, v_hat)
// with its measurement normals too); its workspace path is the polyline through
// the nominal waypoints wp[0..S] plus its deviations; it collides iff a segment
// meets a closed obstacle box (segment_hits_box).
//
// A workgroup takes 64 particles over up to kMcPlans plans.  The deviations do
// not depend on the plan: per kMcChunk steps, three waves (an axis each) run
// the recurrence once and leave it in LDS, with its bounds, and all four then
// take the plans' segments, a wave 64 particles of one.  Lane o first asks
// whether box o can be met by the segment's waypoints plus the bounds; the few
// that can are tested by every particle.  The next chunk's noise is asked for
// before the segments are taken.  It is bound by the chain of steps and by the
// FP64 slab tests: with a wave per plan following the recurrence step by step,
// the noise of a step read only then and every particle against every box, the
// 10,000 particles of an LQG query's smoothing (8 candidates a round, 37 boxes)
// took 193 us a round, now 54.
// ---------------------------------------------------------------------------
constexpr int kMcThreads = 256;
constexpr int kMcParticles = 64;
constexpr int kMcChunk = 16;
constexpr int kMcPlans = 8;

struct McLds {
    double dev[kMcChunk + 1][3][kMcParticles];   // [0]: the step before the chunk
    double lo[3], hi[3];                         // bounds over them
    unsigned long long hit[kMcPlans];
    float obs[kMaxObs * 6];
};

// Plans 0 .. n_p - 1 (at most kMcPlans): wp_of(i) their waypoints, len_of(i)
// their steps (negative: none), count_of(i) where the colliding particles of
// m_base .. m_base + 63 are added.  All threads call it; l.obs holds the boxes.
template <class WpOf, class LenOf, class CountOf>
__device__ __forceinline__ void mc_plans(const SelectArgs& a, int m_base, int n_p, WpOf wp_of, LenOf len_of,
                                         CountOf count_of, McLds& l) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = m_base + lane, M = a.M, n_obs = a.n_obs;
    const bool mine = m < M;
    const unsigned long long all = __ballot(mine);
    const int mr = mine ? m : M - 1;   // (a lane past the end follows the last particle)
    int S = 0;
    for (int i = 0; i < n_p; ++i) S = max(S, len_of(i));
    if (threadIdx.x < kMcPlans) l.hit[threadIdx.x] = 0ull;
    float w0[kMcChunk], w1[kMcChunk], w2[kMcChunk];
    auto load = [&](int s0) {   // the axis's noise of steps s0 .. (read at the last step past the end)
#pragma unroll
        for (int u = 0; u < kMcChunk; ++u) {
            const int s = min(s0 + u, S - 1);
            w0[u] = a.noise_mc[((size_t)s * 6 + 2 * wave) * M + mr];
            w1[u] = a.noise_mc[((size_t)s * 6 + 2 * wave + 1) * M + mr];
            if (a.estimator) w2[u] = a.noise_mc_meas[((size_t)s * 3 + wave) * M + mr];
        }
    };
    double z[4] = {0.0, 0.0, 0.0, 0.0};
    if (wave < 3) {
        l.dev[kMcChunk][wave][lane] = 0.0;
        if (S > 0) load(0);
    }
    for (int c0 = 0; c0 < S; c0 += kMcChunk) {
        if (wave < 3) {
            const double before = l.dev[kMcChunk][wave][lane];   // (this lane's own)
            l.dev[0][wave][lane] = before;
            double lo = before, hi = before;
            bool nan = !(before == before);
#pragma unroll
            for (int u = 0; u < kMcChunk; ++u) {
                if (a.estimator) {
                    lqg_step(a.lqg, z, (double)w0[u], (double)w1[u], (double)w2[u]);
                } else {
                    const double n0 = (double)w0[u], n1 = (double)w1[u];
                    const double pn = a.Acl[0] * z[0] + a.Acl[1] * z[1] + a.L[0] * n0;
                    const double vn = a.Acl[2] * z[0] + a.Acl[3] * z[1] + (a.L[2] * n0 + a.L[3] * n1);
                    z[0] = pn;
                    z[1] = vn;
                }
                l.dev[u + 1][wave][lane] = z[0];
                lo = fmin(lo, z[0]);
                hi = fmax(hi, z[0]);
                nan |= !(z[0] == z[0]);
            }
            for (int o = 32; o > 0; o >>= 1) {
                lo = fmin(lo, __shfl_xor(lo, o, 64));
                hi = fmax(hi, __shfl_xor(hi, o, 64));
            }
            nan = __ballot(nan) != 0ull;   // (a NaN passes the comparisons of its axis)
            if (lane == 0) {
                l.lo[wave] = nan ? -INFINITY : lo;
                l.hi[wave] = nan ? INFINITY : hi;
            }
            if (c0 + kMcChunk < S) load(c0 + kMcChunk);
        }
        __syncthreads();
        for (int i = wave; i < n_p * kMcChunk; i += kMcThreads / 64) {
            const int f = i / kMcChunk, u = i % kMcChunk, s = c0 + u;
            if (s >= len_of(f) || l.hit[f] == all) continue;
            const double* wp = wp_of(f) + (size_t)s * 3;
            double prev[3], cur[3], lo[3], hi[3];
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const double p0 = wp[ax], p1 = wp[3 + ax];
                prev[ax] = p0 + l.dev[u][ax][lane];
                cur[ax] = p1 + l.dev[u + 1][ax][lane];
                // (widened by more than the rounding of the sums)
                lo[ax] = fmin(p0, p1) + l.lo[ax];
                hi[ax] = fmax(p0, p1) + l.hi[ax];
                lo[ax] -= 1e-12 * (1.0 + fabs(lo[ax]));
                hi[ax] += 1e-12 * (1.0 + fabs(hi[ax]));
            }
            bool hit = false;
            for (int o0 = 0; o0 < n_obs; o0 += 64) {
                bool near = false;
                if (o0 + lane < n_obs) {
                    const float* b = l.obs + (o0 + lane) * 6;
                    near = !((hi[0] < (double)b[0]) | (lo[0] > (double)b[3]) | (hi[1] < (double)b[1]) |
                             (lo[1] > (double)b[4]) | (hi[2] < (double)b[2]) | (lo[2] > (double)b[5]));
                }
                unsigned long long some = __ballot(near);
                while (some) {
                    const int o = o0 + __ffsll((long long)some) - 1;
                    some &= some - 1ull;
                    if (!hit) hit = segment_hits_box(prev, cur, l.obs + o * 6);
                }
            }
            const unsigned long long h = __ballot(hit && mine);
            if (lane == 0 && h) atomicOr(&l.hit[f], h);
        }
        __syncthreads();
    }
    __syncthreads();
    if (threadIdx.x < n_p) {
        const int h = (int)__popcll(l.hit[threadIdx.x]);
        if (h && len_of(threadIdx.x) >= 0) atomicAdd(count_of(threadIdx.x), h);
    }
    __syncthreads();
}

// Front plans row, row + rows, ... of n (their waypoints, steps and counts in a).
__device__ __forceinline__ void mc_front(const SelectArgs& a, int m_base, int n, int row, int rows, McLds& l) {
    for (int t = threadIdx.x; t < a.n_obs * 6; t += kMcThreads) l.obs[t] = a.obs[t];
    __syncthreads();
    for (int f0 = row; f0 < n; f0 += rows * kMcPlans) {
        const int n_p = min(kMcPlans, (n - f0 + rows - 1) / rows);
        mc_plans(
            a, m_base, n_p, [&](int i) { return a.wp + (size_t)(f0 + i * rows) * (a.S_max + 1) * 3; },
            [&](int i) { return a.wp_len[f0 + i * rows]; }, [&](int i) { return &a.mc_counts[f0 + i * rows]; }, l);
    }
}

}  // namespace pump
