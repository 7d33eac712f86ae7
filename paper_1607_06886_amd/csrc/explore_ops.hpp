// Per-element operations of one Explore round (Alg. 4), shared by the
// single-query kernels (one launch per phase, whole device) and the batched
// engine (one workgroup per query).  Both drivers run these same bodies, in
// the same orders, so they produce identical plan stores.
#pragma once

#include "device_math.hpp"
#include "pump_internal.hpp"

namespace pump {

__device__ __forceinline__ double stair_get(const unsigned long long* st, int w, int x, int c) {
    return __longlong_as_double((long long)st[(size_t)x * w + c]);
}

// The same entry read with an agent-scope atomic load: current even where
// this XCD's L2 still holds the line from before other workgroups' atomic
// minima (no cache invalidation in between).
__device__ __forceinline__ double stair_get_coherent(const unsigned long long* st, int w, int x,
                                                     int c) {
    unsigned long long* p = const_cast<unsigned long long*>(st) + (size_t)x * w + c;
    return __longlong_as_double(
        (long long)__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

__device__ __forceinline__ unsigned long long lanemask_lt(int lane) {
    return lane ? ((1ull << lane) - 1ull) : 0ull;
}

__device__ __forceinline__ bool boxes_overlap(const float* lo3, const float* hi3, const float* b) {
    return (lo3[0] <= b[3]) & (hi3[0] >= b[0]) & (lo3[1] <= b[4]) & (hi3[1] >= b[1]) &
           (lo3[2] <= b[5]) & (hi3[2] >= b[2]);
}

// Root plan and empty staircases (Alg. 4 first lines).  `t0`/`stride`
// distribute the staircase fill; the root itself is written by thread t0 == 0.
__device__ __forceinline__ void explore_init_fill(const RoundArgs& a, int n_nodes, size_t t0,
                                                  size_t stride) {
    const size_t n = (size_t)n_nodes * a.stair_w;
    for (size_t t = t0; t < n; t += stride) a.stair[t] = 0x7FF0000000000000ull;
}

__device__ __forceinline__ void explore_init_root(const RoundArgs& a, int N) {
    const int W = N / 32;
    a.p_head[0] = 0;
    a.p_parent[0] = -1;
    a.p_edge[0] = -1;
    a.p_step[0] = 0;
    a.p_pop[0] = 0;
    a.p_round[0] = 0;
    a.p_cost[0] = 0.0;
    a.p_state[0] = kOpen;
    for (int w = 0; w < W; ++w) a.p_mask[w] = 0u;
    for (int c = 0; c < a.c_cut && c < a.stair_w; ++c) a.stair[c] = 0ull;  // 0.0 bits
    a.open_out[0] = 0;  // the initial open list is written to open_out
    a.o_inB[0] = 1;
    a.b_ids[0] = 0;
    const int deg = a.row_ptr[1] - a.row_ptr[0];
    a.b_off[0] = 0;
    a.b_off[1] = deg;
    Ctl* c = a.ctl;
    c->n_plans = 1;
    c->n_open = 1;
    c->n_B = 1;
    c->n_pairs = deg;
    c->i = 0;
    c->goal_stop = (a.goal[0] && 0 < a.c_min) ? 1 : 0;
    c->done = c->goal_stop;
    c->err = 0;
    c->n_tasks = 0;
    c->wide = 0;
    c->simulated = c->preprune = c->inserted = c->dropped_steps = c->flagged = 0;
    c->sim_waypoints = c->sim_box_tests = 0;
}

// Group of pair q = tile + lane of the wave: the largest g < n_B with
// b_off[g] <= q (b_off nondecreasing, b_off[0] = 0 <= tile < n_pairs =
// b_off[n_B]).  The wave searches together: 64-way steps (one load per lane
// and a ballot each) narrow the groups down to a window of 64 that holds the
// tile's first pair, one more load brings the window's offsets into the
// lanes, and each lane counts the offsets <= q with a binary search over the
// lanes.  Only a lane whose pair lies past the window (a tile spanning more
// than 64 groups, i.e. groups of degree 0 or 1) searches on in memory.  All
// lanes must call this together.
__device__ __forceinline__ int wave_group_of(const int32_t* __restrict__ b_off, int n_B, int tile,
                                             int q) {
    const int lane = threadIdx.x & 63;
    int lo = 0, hi = n_B;                  // b_off[lo] <= tile, and tile < b_off[hi] or hi = n_B
    while (hi - lo > 64) {
        const int step = (hi - lo + 63) >> 6;
        const int idx = lo + lane * step;
        const unsigned long long le = __ballot(idx < hi && b_off[idx] <= tile);
        const int j = 63 - __clzll((long long)le);   // lane 0 always qualifies
        lo += j * step;
        hi = min(hi, lo + step);
    }
    const int idx = lo + 1 + lane;
    const int v = idx < n_B ? b_off[idx] : INT_MAX;
    int cnt = 0;                           // lanes j with v_j <= q (a prefix of the lanes)
    for (int s = 32; s >= 1; s >>= 1) {
        const int vv = __shfl(v, cnt + s - 1, 64);
        if (vv <= q) cnt += s;
    }
    if (cnt == 63 && __shfl(v, 63, 64) <= q) {
        int l2 = lo + 64, h2 = n_B;        // b_off[l2] <= q < b_off[h2]
        while (h2 - l2 > 1) {
            const int mid = (l2 + h2) >> 1;
            if (b_off[mid] <= q) l2 = mid; else h2 = mid;
        }
        return l2;
    }
    return lo + cnt;
}

// ---------------------------------------------------------------------------
// RemoveDominated (Sec. IV): remove every open plan p for which some plan d
// with the same head has d.cost < p.cost and d.cp_hat <= p.cp_hat.  Per node
// the library keeps the staircase M_x(c) = min{cost of plans in P(x) with
// pop <= c}; p is dominated iff M_{p.head}(p.pop) < p.cost.  Plans removed as
// dominated never change M (their dominator is counted with a lower cost), so
// M needs only insertions: one atomic minimum per kept candidate and level.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void stair_update_pair(const RoundArgs& a, int q) {
    if (a.c_flag[q] != 1) return;
    const int x = a.c_head[q];
    const unsigned long long bits = (unsigned long long)__double_as_longlong(a.c_cost[q]);
    for (int c = a.c_pop[q]; c < a.c_cut; ++c) atomicMin(&a.stair[(size_t)x * a.stair_w + c], bits);
}

// Candidate q: dominated -> flag 2; scan input = survivor.  Returns whether q
// was kept before the test (counts toward `inserted`).  kCoherent: read the
// staircase with atomic loads (the team loop, whose barrier after the
// staircase update does not invalidate the caches).
template <bool kCoherent = false>
__device__ __forceinline__ bool mark_pair(const RoundArgs& a, int t) {
    uint8_t f = a.c_flag[t];
    bool kept = false;
    if (f == 1) {
        kept = true;
        const int x = a.c_head[t], c = a.c_pop[t];
        const double m = kCoherent ? stair_get_coherent(a.stair, a.stair_w, x, c)
                                   : stair_get(a.stair, a.stair_w, x, c);
        if (m < a.c_cost[t]) {
            f = 2;
            a.c_flag[t] = 2;
        }
    }
    a.c_pos[t] = (f == 1) ? 1 : 0;
    return kept;
}

// Open entry i: removed if dominated, closed if in B (P_open \ B), else kept.
template <bool kCoherent = false>
__device__ __forceinline__ void mark_open(const RoundArgs& a, int i) {
    const int p = a.open_in[i];
    const int x = a.p_head[p], c = a.p_pop[p];
    const double m = kCoherent ? stair_get_coherent(a.stair, a.stair_w, x, c)
                               : stair_get(a.stair, a.stair_w, x, c);
    const bool dom = m < a.p_cost[p];
    const bool inB = a.o_inB[i] != 0;
    const uint8_t stt = dom ? kRemoved : (inB ? kClosed : kOpen);
    a.p_state[p] = stt;
    a.o_keep[i] = (stt == kOpen) ? 1 : 0;
}

// Compaction: survivors are appended to the plan store in pair order after
// the kept open plans (c_pos / o_keep hold exclusive scans).
template <int W>
__device__ __forceinline__ void compact_pair(const RoundArgs& a, int t, int n_plans, int n_keep,
                                             int i_round) {
    if (a.c_flag[t] != 1) return;
    const int r = a.c_pos[t];
    const int id = n_plans + r;
    a.p_head[id] = a.c_head[t];
    a.p_parent[id] = a.c_parent[t];
    a.p_edge[id] = a.c_edge[t];
    a.p_step[id] = a.c_step[t];
    a.p_pop[id] = a.c_pop[t];
    a.p_round[id] = i_round;
    a.p_cost[id] = a.c_cost[t];
    a.p_state[id] = kOpen;
    for (int w = 0; w < W; ++w) a.p_mask[(size_t)id * W + w] = a.c_mask[(size_t)t * W + w];
    a.open_out[n_keep + r] = id;
}

__device__ __forceinline__ void compact_open(const RoundArgs& a, int i) {
    const int p = a.open_in[i];
    if (a.p_state[p] == kOpen) a.open_out[a.o_keep[i]] = p;
}

// After compaction (one thread): publish the new counts; err on overflow.
__device__ __forceinline__ void compact_finalize(Ctl* c, int64_t cap) {
    const int n_surv = c->scan_total[0];
    const int n_keep = c->scan_total[1];
    if ((long long)c->n_plans + n_surv > cap) {
        c->err = 1;
        c->done = 1;
        c->n_surv = n_surv;   // the plan store needs n_plans + n_surv entries
        return;
    }
    c->n_plans += n_surv;
    c->n_open = n_keep + n_surv;
    c->min_cost_bits = 0x7FF0000000000000ull;
    c->goal_stop = 0;
}

// Next group (one thread): i <- i + 1; when that group would be empty the
// loop only advances i, so i jumps to the first value admitting the cheapest
// open plan (cost <= i lambda r_n).
__device__ __forceinline__ void pick_next_i(Ctl* c, double h) {
    if (c->err) return;
    if (c->n_open == 0) {
        c->done = 1;
        c->i = c->i + 1;
        return;
    }
    const double mc = __longlong_as_double((long long)c->min_cost_bits);
    if (!(mc >= 0.0 && mc < 1e300) || !(mc / h < 2.0e9)) {  // no finite cheapest open plan
        c->err = 3;
        c->done = 1;
        return;
    }
    long long k = (long long)ceil(mc / h);
    if (k < 0) k = 0;
    while (k > 0 && mc <= (double)(k - 1) * h) --k;
    while (!(mc <= (double)k * h)) ++k;
    const long long inext = c->i + 1;
    c->i = (int)(k > inext ? k : inext);
}

// Open entry i of the new list: in B?  (scan input in o_keep).  Returns
// whether it stops the loop (a goal plan of B with cp_hat < alpha_min).
__device__ __forceinline__ bool flag_group_one(const RoundArgs& a, int i, double thr) {
    const int p = a.open_out[i];
    const bool inB = a.p_cost[p] <= thr;
    a.o_inB[i] = inB ? 1 : 0;
    a.o_keep[i] = inB ? 1 : 0;
    return inB && a.goal[a.p_head[p]] && a.p_pop[p] < a.c_min;
}

__device__ __forceinline__ void scatter_group_one(const RoundArgs& a, int i) {
    if (a.o_inB[i]) a.b_ids[a.o_keep[i]] = a.open_out[i];
}

}  // namespace pump
