// Expansion of Explore's pairs for the box model (Alg. 4: Steer, Propagate,
// Collide, Cost, CP cutoff), one pair per lane from its edge to its particle
// bits.
//
// A workgroup takes its pairs a pass at a time.  pair_front settles the
// pairs whose fate their parent and the staircases decide (past S_max,
// already dominated) and hands the others on as records in LDS, so that the
// geometry behind it runs on full waves although only some tenths of the
// pairs reach it.  pair_particles marks a record's waypoints where the
// particle cloud can meet a box, then takes the marked ones in order: each
// box's hits come from the rank tables (rank_tables.hpp), a few lane
// operations per face instead of a test per particle.  Wide records, whose
// clouds meet many boxes, are tested by particle all the same (by_particle),
// by their workgroup or, where many are wide, from a queue all workgroups share.
//
// Measured on the 20,000-sample indoor query (N = 256, 60 boxes; 1.0e7 pairs,
// 9.5e6 tested waypoints, 1.1e7 box tests): expansion took 5.5 ms as a pair
// kernel and a particle kernel with a wave per pair and a test per particle
// (3.9 ms, bound by VALU issue), and takes 2.1 to 2.3 ms here.  What bounds it is
// latency: its waves wait some 60 % of their cycles on the chains of gathers,
// at three waves per SIMD (158 registers for N = 256).
#pragma once

#include "box_bins.hpp"
#include "explore_ops.hpp"
#include "rank_tables.hpp"

namespace pump {

struct PairRec {
    double tau, cost;
    int32_t sl;                // candidate slot
    int32_t p;                 // parent plan
    uint32_t nodes;            // edge endpoints: head | x << 16 (node ids < 65536)
    int32_t ks;                // waypoints K on the edge (at most 32) | parent's steps << 8
};
static_assert(sizeof(PairRec) == 32, "PairRec is two 16-byte LDS words");

// Counters of one wave over a pass (the same in every lane: sums of ballots), and
// a workgroup's totals, in LDS: a workgroup may carry a whole query, whose
// waypoints and box tests go past 32 bits (2^26 pairs a round, 32 waypoints each,
// up to 256 boxes at each).
struct PairCounts {
    int sim = 0, pre = 0, drop = 0, wp = 0, bt = 0, flag = 0;
};
struct PairTotals {
    unsigned long long sim, pre, drop, wp, bt, flag;
};
// (of a pass's at most 1024 records; a few more are carried over)
static_assert(2048ll * kMaxWaypoints * kMaxObs < (1ll << 31), "a pass's counts fit 32 bits");

// A wave's counters to the totals; they start over.
__device__ __forceinline__ void add_counts(PairTotals* tot, PairCounts& n) {
    if ((threadIdx.x & 63) == 0) {
        if (n.sim) atomicAdd(&tot->sim, (unsigned long long)n.sim);
        if (n.pre) atomicAdd(&tot->pre, (unsigned long long)n.pre);
        if (n.drop) atomicAdd(&tot->drop, (unsigned long long)n.drop);
        if (n.wp) atomicAdd(&tot->wp, (unsigned long long)n.wp);
        if (n.bt) atomicAdd(&tot->bt, (unsigned long long)n.bt);
        if (n.flag) atomicAdd(&tot->flag, (unsigned long long)n.flag);
    }
    n = PairCounts();
}

__device__ __forceinline__ int lanes_of(bool b) { return (int)__popcll(__ballot(b)); }

enum PairFate : int { kPairGoes = 0, kPairDropped = 1, kPairDominated = 2, kPairNone = 3 };

// The boxes in dynamic LDS: raw faces, faces grown by the guard band, centres and
// half extents shrunk by it (c xyz, h - kGuard xyz; their rounding is far below
// the band), bins.
struct BoxLds {
    const float* raw;
    const float* out;
    const float* in;
    BinView bins;
    int n_obs;
};

__host__ __device__ constexpr size_t box_lds_bytes(int n_obs) {
    return (size_t)(18 * n_obs + bin_words(n_obs) + 2) * 4;
}

// Fill by the whole workgroup; a barrier must follow before use.
__device__ __forceinline__ BoxLds stage_box_lds(const RoundArgs& a, char* mem) {
    BoxLds s;
    const int n_obs = a.n_obs, nw = (n_obs + 63) / 64;
    uint32_t* set = reinterpret_cast<uint32_t*>(mem);
    const int n_set = bin_words(n_obs) - kBinHeader;
    float* raw = reinterpret_cast<float*>(set + n_set);
    float* out = raw + 6 * n_obs;
    float* in = out + 6 * n_obs;
    for (int t = threadIdx.x; t < n_set; t += blockDim.x) set[t] = a.bins[kBinHeader + t];
    for (int t = threadIdx.x; t < 6 * n_obs; t += blockDim.x) {
        const float v = a.obs[t];
        const bool is_lo = t % 6 < 3;
        raw[t] = v;
        out[t] = is_lo ? v - kGuard : v + kGuard;
        const float lo = is_lo ? v : a.obs[t - 3], hi = is_lo ? a.obs[t + 3] : v;
        in[t] = is_lo ? 0.5f * (lo + hi) : 0.5f * (hi - lo) - kGuard;
    }
    for (int k = 0; k < 3; ++k) {
        s.bins.org[k] = __uint_as_float(a.bins[k]);
        s.bins.scale[k] = __uint_as_float(a.bins[3 + k]);
    }
    s.bins.set = reinterpret_cast<const unsigned long long*>(set);
    s.bins.nw = nw;
    s.raw = raw;
    s.out = out;
    s.in = in;
    s.n_obs = n_obs;
    return s;
}

// Pair q of group lo (wave_group_of): identity, edge and parent plan to
// candidate slot q - a.q0; its record, unless it is settled here (dropped past
// S_max, or dominated at x already by the parent's own count).
__device__ __forceinline__ PairFate pair_front(const RoundArgs& a, int q, int lo, PairRec& r) {
    const int p = a.b_ids[lo];
    const int head = a.p_head[p];
    const int e = a.row_ptr[head] + (q - a.b_off[lo]);
    const int x = a.col[e];
    const int sl = q - a.q0;
    a.c_parent[sl] = p;   // every formed pair records its identity
    a.c_head[sl] = x;
    const double tau = a.etau[e];
    const double cost = a.p_cost[p] + a.ecost[e];
    const int K = max(1, (int)ceil(tau / a.dt));
    const int s_p = a.p_step[p];
    if (s_p + K > a.S_max) {
        a.c_flag[sl] = 0;
        a.c_pop[sl] = -2;
        return kPairDropped;
    }
    if (a.preprune && stair_get(a.stair, a.stair_w, x, a.p_pop[p]) < cost) {
        a.c_flag[sl] = 0;
        a.c_pop[sl] = -1;
        return kPairDominated;
    }
    a.c_edge[sl] = e;
    a.c_cost[sl] = cost;
    a.c_step[sl] = s_p + K;
    r = PairRec{tau, cost, sl, p, (uint32_t)head | ((uint32_t)x << 16), K | (s_p << 8)};
    return kPairGoes;
}

__device__ __forceinline__ void load_state(const float* __restrict__ X, uint32_t v, float* x) {
    const float2* p = reinterpret_cast<const float2*>(X + (size_t)v * 6);
    const float2 a = p[0], b = p[1], c = p[2];
    x[0] = a.x; x[1] = a.y; x[2] = b.x; x[3] = b.y; x[4] = c.x; x[5] = c.y;
}

// The N-bit set of a prefix row, W words.
template <int W>
__device__ __forceinline__ void load_set(const uint32_t* __restrict__ m, uint32_t (&v)[W]) {
    if constexpr (W >= 4) {
#pragma unroll
        for (int i = 0; i < W / 4; ++i) {
            const uint4 u = reinterpret_cast<const uint4*>(m)[i];
            v[4 * i] = u.x; v[4 * i + 1] = u.y; v[4 * i + 2] = u.z; v[4 * i + 3] = u.w;
        }
    } else if constexpr (W == 2) {
        const uint2 u = *reinterpret_cast<const uint2*>(m);
        v[0] = u.x; v[1] = u.y;
    } else {
        v[0] = m[0];
    }
}

template <int W>
__device__ __forceinline__ void store_set(uint32_t* __restrict__ m, const uint32_t (&v)[W]) {
    if constexpr (W >= 4) {
#pragma unroll
        for (int i = 0; i < W / 4; ++i)
            reinterpret_cast<uint4*>(m)[i] = make_uint4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
    } else if constexpr (W == 2) {
        *reinterpret_cast<uint2*>(m) = make_uint2(v[0], v[1]);
    } else {
        m[0] = v[0];
    }
}

// Cloud row of a step, and the particle cloud's box (FP32) around a nominal
// point (FP64).
__device__ __forceinline__ void load_cloud(const float* __restrict__ cl, float* c6) {
    const float2* p = reinterpret_cast<const float2*>(cl);
    const float2 u = p[0], v = p[1], w = p[2];
    c6[0] = u.x; c6[1] = u.y; c6[2] = v.x; c6[3] = v.y; c6[4] = w.x; c6[5] = w.y;
}

__device__ __forceinline__ void cloud_box(const double* nom, const float* c6, float* lo3, float* hi3) {
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const float n32 = (float)nom[ax];
        lo3[ax] = n32 + c6[ax] - 1e-6f;
        hi3[ax] = n32 + c6[3 + ax] + 1e-6f;
    }
}

__device__ __forceinline__ void waypoint_box(const Cubic* cs, double t, const float* __restrict__ cl,
                                             double* nom, float* c6, float* lo3, float* hi3) {
    load_cloud(cl, c6);
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) nom[ax] = cs[ax].at(t);
    cloud_box(nom, c6, lo3, hi3);
}

// The cubics of a record's edge and its waypoint spacing.
__device__ __forceinline__ double record_cubics(const RoundArgs& a, const PairRec& rec, Cubic* cs) {
    float x0[6], x1[6];
    load_state(a.X, rec.nodes & 0xFFFFu, x0);
    load_state(a.X, rec.nodes >> 16, x1);
    hermite_r(x0, x1, rec.tau, recip_fast(rec.tau), cs);
    return rec.tau * recip_fast((double)(rec.ks & 255));
}

// Particle decisions of a pair that lie within kFlagEps of a box face: those
// of particles the parent has not lost, near some face at a marked waypoint
// and inside no box by more than kFlagEps there.  One pair by the whole wave
// (wave-uniform arguments), particles l, l + 64, ... on lane l; the pair's
// cutoff has not been reached, so every marked waypoint counts.  close: the
// marked waypoints where a face has a particle within kFlagEps.  Mostly such a
// particle lies far outside the box on another axis, so those waypoints are taken
// first, and the others only if a particle stays.
template <int N>
__device__ __forceinline__ int flagged_count(const RoundArgs& a, const PairRec& rec, uint32_t near,
                                             uint32_t close, const BoxLds& s) {
    constexpr int W = N / 32, PPL = N >= 64 ? N / 64 : 1;
    const int lane = threadIdx.x & 63;
    const int j0 = N >= 64 ? lane : (lane & (N - 1));
    const int s_p = rec.ks >> 8, p = rec.p;
    Cubic cs[3];
    const double dtk = record_cubics(a, rec, cs);
    uint32_t nm = 0u, dm = 0u;
    bool rest = false;   // past the close waypoints
    for (uint32_t m = near & close; m || !rest; m &= m - 1u) {
        if (!m) {
            if (__ballot(nm != 0u) == 0ull) return 0;
            rest = true;
            m = near & ~close;
            if (!m) break;
        }
        const int k = __ffs((int)m), st = s_p + k;
        double nom[3];
        float c6[6], lo3[3], hi3[3];
        waypoint_box(cs, (double)k * dtk, a.cloud + (size_t)st * 6, nom, c6, lo3, hi3);
        float d[PPL][3];
#pragma unroll
        for (int ax = 0; ax < 3; ++ax)
#pragma unroll
            for (int r = 0; r < PPL; ++r) d[r][ax] = a.D[((size_t)st * 3 + ax) * N + r * 64 + j0];
        for (int c0 = 0; c0 < s.n_obs; c0 += 64) {
            const int o = c0 + lane;
            unsigned long long om =
                __ballot(o < s.n_obs && boxes_overlap(lo3, hi3, s.out + o * 6));
            while (om) {
                const float* b = s.raw + (c0 + __ffsll((long long)om) - 1) * 6;
                om &= om - 1ull;
#pragma unroll
                for (int r = 0; r < PPL; ++r) {
                    double dmin = INFINITY;
                    bool ok = true;
#pragma unroll
                    for (int ax = 0; ax < 3; ++ax) {
                        const double yy = nom[ax] + (double)d[r][ax];
                        ok &= yy == yy;
                        dmin = fmin(dmin, fmin(yy - (double)b[ax], (double)b[3 + ax] - yy));
                    }
                    if (ok && dmin >= kFlagEps) dm |= 1u << r;
                    if (ok && fabs(dmin) < kFlagEps) nm |= 1u << r;
                }
            }
        }
    }
    const uint32_t f = nm & ~dm;
    int n = 0;
#pragma unroll
    for (int r = 0; r < PPL; ++r) {
        const unsigned long long fb = __ballot((N >= 64 || lane < N) && ((f >> r) & 1u));
        n += __popc((uint32_t)fb & ~a.p_mask[(size_t)p * W + 2 * r]);
        if (N >= 64) n += __popc((uint32_t)(fb >> 32) & ~a.p_mask[(size_t)p * W + 2 * r + 1]);
    }
    return n;
}

// Lane k's value in every lane (k wave-uniform).
__device__ __forceinline__ int lane_int(int v, int k) { return __builtin_amdgcn_readlane(v, k); }
__device__ __forceinline__ float lane_float(float v, int k) { return __int_as_float(lane_int(__float_as_int(v), k)); }
__device__ __forceinline__ double lane_double(double v, int k) {
    const long long b = __double_as_longlong(v);
    const int lo = lane_int((int)(unsigned)(b & 0xFFFFFFFFll), k), hi = lane_int((int)(b >> 32), k);
    return __longlong_as_double(((long long)(unsigned)hi << 32) | (unsigned)lo);
}

// ---------------------------------------------------------------------------
// A record by the whole wave, particles across its lanes (lane l has particles
// l, l + 64, ..., so the hits of particle row r are one ballot): at each marked
// waypoint every particle against the boxes that the cloud meets, in FP32 with an
// FP64 re-test inside the guard band, until the pair reaches the cutoff.  The next
// waypoint's deviations are asked for before a waypoint is tested, and the clouds of
// all of them at the start where the registers are there (N < 256: a load and its
// wait less for each); with 32 particles the halves of the wave take the boxes in
// turn (1000 samples, 50 boxes, sigma 0.2, alpha 0.9, N = 32: 4.7 ms without the
// two, 3.8 with them).
//
// For wide records.  A rank test takes a lane three dependent gathers for each face
// that cuts the cloud; where a cloud is wider than a box that is most of its six
// faces, and the lanes of a wave differ in how many boxes they have.  A test by
// particle is some 14 instructions of the wave for each box and 64 particles.
// kWideBoxes, the boxes a marked waypoint's bins hold on average from which a record
// is wide: with 1, 2, 3, 4, 6 and 10, a query with 4.2 boxes a waypoint (3000
// samples, 60 boxes, 256 particles, sigma 0.08, alpha 0.3) took 13.1, 13.2, 13.2,
// 13.6, 15.0 and 17.2 ms, one with 1.2 (8000-sample indoor, sigma 0.02) 3.6, 2.8,
// 2.5, 2.5, 2.5 and 2.5.
//
// A round's wide records lie together (pairs of the same plans), so that some
// workgroups had far more of them than others.  Where half of a round's marked
// records were wide (Ctl::wide), the next round's go through a queue that the whole
// device shares, all of them, since a few left to the rank test would end last:
// that query then takes 8.1 ms, and with sigma 0.2 (18 boxes a waypoint) 6.9 where
// the rank test alone took 27.5.  Other rounds are spared the further launch or
// barrier.
// ---------------------------------------------------------------------------
template <int N>
__device__ __forceinline__ void by_particle(const RoundArgs& a, const BoxLds& s, const PairRec& rec, uint32_t near,
                                            PairCounts& n) {
    constexpr int W = N / 32, PPL = N >= 64 ? N / 64 : 1;
    const int lane = threadIdx.x & 63;
    const bool valid = N >= 64 || lane < N;
    const int j0 = N >= 64 ? lane : (lane & (N - 1));
    constexpr bool kHalves = N < 64;      // each half of the wave takes every other box
    constexpr bool kCloudsHeld = N < 256; // (its registers are all taken)
    const int s_p = rec.ks >> 8;
    uint32_t wm = near;
    float d[PPL][3], dn[PPL][3];
    auto ask = [&](int k) {
#pragma unroll
        for (int ax = 0; ax < 3; ++ax)
#pragma unroll
            for (int r = 0; r < PPL; ++r) dn[r][ax] = a.D[((size_t)(s_p + k) * 3 + ax) * N + r * 64 + j0];
    };
    ask(__ffs((int)wm));
    // lane k - 1 holds waypoint k's nominal point and cloud box
    double my_nom[3];
    float my_lo[3], my_hi[3];
    {
        float c6[6];
        if (kCloudsHeld) load_cloud(a.cloud + (size_t)(s_p + min(lane + 1, rec.ks & 255)) * 6, c6);
        Cubic cs[3];
        const double dtk = record_cubics(a, rec, cs);
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) my_nom[ax] = cs[ax].at((double)(lane + 1) * dtk);
        if (kCloudsHeld) cloud_box(my_nom, c6, my_lo, my_hi);
    }
    uint32_t par = 0u;   // the parent's bits of this lane's particles
#pragma unroll
    for (int r = 0; r < PPL; ++r) {
        const int j = r * 64 + j0;
        par |= ((a.p_mask[(size_t)rec.p * W + (j >> 5)] >> (j & 31)) & 1u) << r;
    }
    if (!valid) par = 0u;
    uint32_t hm = 0u, dm = 0u, nm = 0u;   // per particle r: hit, deep, near a face
    for (;;) {
        const int k = __ffs((int)wm);
        wm &= wm - 1u;
#pragma unroll
        for (int r = 0; r < PPL; ++r)
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) d[r][ax] = dn[r][ax];
        if (wm) ask(__ffs((int)wm));
        ++n.wp;
        double nom[3];
        float lo3[3], hi3[3];
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) nom[ax] = lane_double(my_nom[ax], k - 1);
        if (kCloudsHeld) {
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                lo3[ax] = lane_float(my_lo[ax], k - 1);
                hi3[ax] = lane_float(my_hi[ax], k - 1);
            }
        } else {
            float c6[6];
            load_cloud(a.cloud + (size_t)(s_p + k) * 6, c6);
            cloud_box(nom, c6, lo3, hi3);
        }
        float y[PPL][3];
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            const float n32 = (float)nom[ax];
#pragma unroll
            for (int r = 0; r < PPL; ++r) y[r][ax] = n32 + d[r][ax];
        }
        for (int c0 = 0; c0 < s.n_obs; c0 += 64) {
            const int o = c0 + lane;
            unsigned long long om = __ballot(o < s.n_obs && boxes_overlap(lo3, hi3, s.out + o * 6));
            n.bt += (int)__popcll(om);
            while (om) {
                int ob = c0 + __ffsll((long long)om) - 1;
                om &= om - 1ull;
                if (kHalves && om) {
                    if (lane >= N) ob = c0 + __ffsll((long long)om) - 1;
                    om &= om - 1ull;
                }
                // u = max over axes of |y - c| - (h - g): u <= 0, inside by more
                // than the guard band (a hit, deep); 0 < u <= 2 g, within it,
                // decided in FP64 (rare)
                const float* bc = s.in + ob * 6;
                const float cx = bc[0], cy = bc[1], cz = bc[2], hx = bc[3], hy = bc[4], hz = bc[5];
                uint32_t inb = 0u, bnd = 0u;
#pragma unroll
                for (int r = 0; r < PPL; ++r) {
                    const float u = fmaxf(fmaxf(fabsf(y[r][0] - cx) - hx, fabsf(y[r][1] - cy) - hy),
                                          fabsf(y[r][2] - cz) - hz);
                    inb |= (u <= 0.0f ? 1u : 0u) << r;
                    bnd |= (u > 0.0f && u <= 2.0f * kGuard ? 1u : 0u) << r;
                }
                hm |= inb;
                dm |= inb;
                if (!valid && !kHalves) bnd = 0u;
                if (__ballot(bnd != 0u) == 0ull) continue;
                const float* b = s.raw + ob * 6;
#pragma unroll
                for (int r = 0; r < PPL; ++r) {
                    if (!(bnd & (1u << r))) continue;
                    double dmin = INFINITY;
#pragma unroll
                    for (int ax = 0; ax < 3; ++ax) {
                        // (kept in this branch: without the empty asm the compiler
                        // takes these FP64 sums before the box loop, for every
                        // waypoint)
                        float dv = d[r][ax];
                        asm volatile("" : "+v"(dv));
                        const double yy = nom[ax] + (double)dv;
                        dmin = fmin(dmin, fmin(yy - (double)b[ax], (double)b[3 + ax] - yy));
                    }
                    if (dmin >= 0.0) hm |= 1u << r;
                    if (dmin >= kFlagEps) dm |= 1u << r;
                    if (fabs(dmin) < kFlagEps) nm |= 1u << r;
                }
            }
        }
        int cnt = 0;
        if (kHalves) hm |= (uint32_t)__shfl_xor((int)hm, N, 64);
#pragma unroll
        for (int r = 0; r < PPL; ++r) cnt += (int)__popcll(__ballot(valid && (((hm | par) >> r) & 1u)));
        if (!wm || cnt >= a.c_cut) break;
    }
    if (kHalves) {
        dm |= (uint32_t)__shfl_xor((int)dm, N, 64);
        nm |= (uint32_t)__shfl_xor((int)nm, N, 64);
    }
    uint32_t words[W];
    int popc = 0, flg = 0;
#pragma unroll
    for (int r = 0; r < PPL; ++r) {
        const unsigned long long hb = __ballot(valid && (((hm | par) >> r) & 1u));
        flg += (int)__popcll(__ballot(valid && (((nm & ~dm & ~par) >> r) & 1u)));
        popc += (int)__popcll(hb);
        words[(2 * r) % W] = (uint32_t)hb;
        if (N >= 64) words[(2 * r + 1) % W] = (uint32_t)(hb >> 32);
    }
    const int sl = rec.sl;
    bool keep = popc < a.c_cut;
    if (keep) n.flag += flg;   // flagged decisions of pairs below the cut
    if (keep && a.preprune && stair_get(a.stair, a.stair_w, (int)(rec.nodes >> 16), popc) < rec.cost) {
        keep = false;
        ++n.pre;
    }
    if (lane == 0) {
        a.c_flag[sl] = keep ? 1 : 0;
        a.c_pop[sl] = popc;
        if (keep) store_set<W>(a.c_mask + (size_t)sl * W, words);
    }
}

// The queue's n_tasks records by the waves of G workgroups (this one is b): each
// wave gathers up to 64 of its records at once, a lane each, from what pair_front
// and mark_pass left in their slots.
template <int N>
__device__ __forceinline__ void queued_by_particle(const RoundArgs& a, int n_tasks, int b, int G, const BoxLds& s,
                                             PairTotals* tot) {
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    const int waves = G * nw, me = b * nw + (threadIdx.x >> 6);
    PairCounts n;
    for (long long base = me; base < n_tasks; base += 64ll * waves) {
        const long long mine = base + (long long)lane * waves;
        PairRec r{0.0, 0.0, 0, 0, 0u, 0};
        int near = 0;
        if (mine < n_tasks) {
            r.sl = a.c_pos[mine];
            near = a.c_pop[r.sl];
            r.p = a.c_parent[r.sl];
            r.cost = a.c_cost[r.sl];
            r.tau = a.etau[a.c_edge[r.sl]];
            r.nodes = (uint32_t)a.p_head[r.p] | (uint32_t)a.c_head[r.sl] << 16;
            const int s_p = a.p_step[r.p];
            r.ks = (a.c_step[r.sl] - s_p) | (s_p << 8);
        }
        const int m = (int)min(64ll, (n_tasks - base + waves - 1) / waves);
        for (int i = 0; i < m; ++i) {
            PairRec rec;
            rec.tau = lane_double(r.tau, i);
            rec.cost = lane_double(r.cost, i);
            rec.sl = lane_int(r.sl, i);
            rec.p = lane_int(r.p, i);
            rec.nodes = (uint32_t)lane_int((int)r.nodes, i);
            rec.ks = lane_int(r.ks, i);
            by_particle<N>(a, s, rec, (uint32_t)lane_int(near, i), n);
        }
        add_counts(tot, n);
    }
}

// Candidate boxes of a waypoint's cloud box, from the bins queried a guard
// band wider than the grown faces.
__device__ __forceinline__ void cloud_bins(const BoxLds& s, const float* lo3, const float* hi3,
                                           BinRange& br) {
    float l[3], h[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        l[ax] = lo3[ax] - 2.0f * kGuard;
        h[ax] = hi3[ax] + 2.0f * kGuard;
    }
    bin_range(s.bins, l, h, br);
}

// First candidate of word w (bits m, consumed) that the cloud box meets, or -1.
__device__ __forceinline__ int next_box(const BoxLds& s, const float* lo3, const float* hi3, int w,
                                        unsigned long long& m) {
    while (m) {
        const int o = w * 64 + __ffsll((long long)m) - 1;
        m &= m - 1ull;
        if (boxes_overlap(lo3, hi3, s.out + o * 6)) return o;
    }
    return -1;
}

// Marked waypoints of a record, those whose cloud box meets an obstacle, among
// waypoints k0, k0 + dk, ...; weight: how many boxes their bins hold (from the
// first word of the sets with one that the cloud meets).
__device__ __forceinline__ uint32_t mark_waypoints(const RoundArgs& a, const PairRec& rec,
                                                   const BoxLds& s, const float* gl, const float* gh,
                                                   int k0, int dk, int& weight) {
    const int K = rec.ks & 255, s_p = rec.ks >> 8;
    const float* cloud = a.cloud + (size_t)s_p * 6;
    float x0[6], x1[6], c6[6];
    load_cloud(cloud + min(k0, K) * 6, c6);
    load_state(a.X, rec.nodes & 0xFFFFu, x0);
    load_state(a.X, rec.nodes >> 16, x1);
    // boxes the cloud can reach anywhere along the edge: the edge lies in the
    // hull of its Bernstein points
    float elo[3], ehi[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const double h3 = rec.tau * (1.0 / 3.0);
        const double p0 = (double)x0[ax], p3 = (double)x1[ax];
        const double p1 = p0 + h3 * (double)x0[3 + ax], p2 = p3 - h3 * (double)x1[3 + ax];
        elo[ax] = (float)fmin(fmin(p0, p3), fmin(p1, p2)) + gl[ax] - (1e-5f + 2.0f * kGuard);
        ehi[ax] = (float)fmax(fmax(p0, p3), fmax(p1, p2)) + gh[ax] + (1e-5f + 2.0f * kGuard);
    }
    BinRange br;
    bin_range(s.bins, elo, ehi, br);
    unsigned long long any = 0ull;
    for (int w = 0; w < s.bins.nw; ++w) any |= bin_candidates(s.bins, br, w);
    if (!any) return 0u;
    Cubic cs[3];
    hermite_r(x0, x1, rec.tau, recip_fast(rec.tau), cs);
    const double dtk = rec.tau * recip_fast((double)K);
    uint32_t near = 0u;
    for (int k = k0; k <= K; k += dk) {
        float cn[6];   // the next waypoint's row, in flight during this one
        load_cloud(cloud + min(k + dk, K) * 6, cn);
        double nom[3];
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) nom[ax] = cs[ax].at((double)k * dtk);
        float lo3[3], hi3[3];
        cloud_box(nom, c6, lo3, hi3);
        cloud_bins(s, lo3, hi3, br);
        bool meets = false;
        for (int w = 0; w < s.bins.nw && !meets; ++w) {
            unsigned long long m = bin_candidates(s.bins, br, w);
            const int held = (int)__popcll(m);
            meets = next_box(s, lo3, hi3, w, m) >= 0;
            weight += meets ? held * (s.bins.nw - w) : 0;
        }
        near |= (meets ? 1u : 0u) << (k - 1);
#pragma unroll
        for (int i = 0; i < 6; ++i) c6[i] = cn[i];
    }
    return near;
}

// One of three values by index, taken by value.
template <class T>
__device__ __forceinline__ T pick3(int i, T a, T b, T c) {
    return i == 0 ? a : (i == 1 ? b : c);
}

typedef double Vec4d __attribute__((ext_vector_type(4)));
typedef float Vec8f __attribute__((ext_vector_type(8)));

template <int W>
__device__ __forceinline__ int set_count(const uint32_t (&v)[W]) {
    int n = 0;
#pragma unroll
    for (int i = 0; i < W; ++i) n += __popc(v[i]);
    return n;
}

// Faces of a box that some particle at the waypoint may lie beyond, or within
// kFlagEps of (bits 0-2 the lower faces, 3-5 the upper ones; every face with
// `all`).
__device__ __forceinline__ int cut_faces(const double* nom, const float* c6, const float* b, bool all) {
    int f = 0;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const bool l = nom[ax] + (double)c6[ax] < (double)b[ax] + 2.0 * kFlagEps;
        const bool h = nom[ax] + (double)c6[3 + ax] > (double)b[3 + ax] - 2.0 * kFlagEps;
        f |= (all || l ? 1 : 0) << ax | (all || h ? 1 : 0) << (3 + ax);
    }
    return f;
}

// Face f of the box: its particles before or past the face leave `hit`.
template <int N>
__device__ __forceinline__ void face_hits(const RoundArgs& a, const BoxLds& s, const double* nom,
                                          const float* c6, int st, int box, int f,
                                          uint32_t (&hit)[N / 32], bool& close) {
    constexpr int W = N / 32;
    const bool upper = f >= 3;
    const int ax = upper ? f - 3 : f;
    const double y = pick3(ax, nom[0], nom[1], nom[2]);
    const RankCells cells(N, pick3(ax, c6[0], c6[1], c6[2]), pick3(ax, c6[3], c6[4], c6[5]));
    const int col = st * 3 + ax;
    const int r = face_rank<N>(a.rank + (size_t)col * rank_row(N), cells, y, (double)s.raw[box * 6 + f],
                               upper, close);
    uint32_t pre[W];
    load_set<W>(a.prefix + ((size_t)col * (N + 1) + r) * W, pre);
    const uint32_t inv = upper ? 0u : 0xFFFFFFFFu;
#pragma unroll
    for (int i = 0; i < W; ++i) hit[i] &= pre[i] ^ inv;
}

// LDS of expand_box_block for a workgroup of T threads.
struct PairLds {
    PairRec* front;            // [2 T] pairs that passed pair_front (a stack)
    PairRec* list;             // [T] records whose particles are tested (from its end:
                               // the wide ones), ...
    uint32_t* near;            // [T] ... and their marked waypoints
    PairRec* mine;             // [T] the record each lane is at
    uint32_t* mine_near;       // [T]
    int* cnt;                  // [6]: stack, list entries, entries taken, the same two of
                               // the wide records, and the share of those (Ctl::wide)
};
constexpr int kPairCounters = 6;
constexpr int pair_lds_bytes(int T) { return T * (4 * (int)sizeof(PairRec) + 8) + 32; }

__device__ __forceinline__ PairLds pair_lds(char* mem, int T) {
    PairLds l;
    l.front = reinterpret_cast<PairRec*>(mem);
    l.list = l.front + 2 * T;
    l.mine = l.list + T;
    l.near = reinterpret_cast<uint32_t*>(l.mine + T);
    l.mine_near = l.near + T;
    l.cnt = reinterpret_cast<int*>(l.mine_near + T);
    return l;
}

// The particles of the listed records, a record per lane and one face of a
// (waypoint, box) test a step.  Records differ by an order of magnitude in
// their waypoints and boxes, and many stop at the cutoff, so every lane runs
// through its own tests and takes the next record as soon as kRefill lanes of
// its wave wait for one.  With `more` records to come a wave leaves its loop
// when the list is empty and fewer than kLow of its lanes are busy; those go on
// with the next list (their state is the caller's).  On the 20,000-sample indoor query a
// step's face search ran on 21 of 64 lanes with every list drained by itself.
// A step is a chain of three dependent gathers (cell, window, prefix set).
//
// A lane's place in its record: nom, c6 the waypoint (step st) and its cloud
// row; wm the marked waypoints left; cand the boxes of the waypoint still to
// test in word cw; box, faces the box it is at and its faces still to search;
// hit that box's hits, acc the parent's bits and the hits so far; close the steps
// (modulo 32) at which a face has a particle within kFlagEps.  (The
// record's fields stay in LDS and the edge's cubic is taken anew at each
// waypoint: with both held, 34 registers more, the kernel spilled.)
//
// Once a pair's count reaches c_cut it is cut whatever its remaining
// waypoints add, so it stops there: a cut pair's count is then some value
// >= c_cut rather than its full count.
template <int N>
__device__ __forceinline__ void test_records(const RoundArgs& a, const BoxLds& s, const PairLds& l,
                                             int n_list, bool more, bool all_faces,
                                             Vec4d& nomv, Vec8f& c6v,
                                             uint32_t (&acc)[N / 32], uint32_t (&hit)[N / 32],
                                             unsigned long long& cand, uint32_t& wm, int& st,
                                             int& box, int& cw, int& faces, bool& active,
                                             uint32_t& close, PairCounts& n) {
    constexpr int W = N / 32;
    constexpr int kRefill = 8, kLow = 40;
    const int lane = threadIdx.x & 63;
    const PairRec& mine = l.mine[threadIdx.x];
    bool left = n_list > 0;
    // (state that outlives the call sits in vector values: held in arrays, the
    // choice of an axis by index below kept them in scratch memory)
    double nom[3] = {nomv.x, nomv.y, nomv.z};
    float c6[6] = {c6v.s0, c6v.s1, c6v.s2, c6v.s3, c6v.s4, c6v.s5};
    // the waypoint's next box the cloud box meets, and its faces that some
    // particle may lie beyond, or within kFlagEps of
    auto advance_box = [&]() {
        float lo3[3], hi3[3];
        cloud_box(nom, c6, lo3, hi3);
        box = next_box(s, lo3, hi3, cw, cand);
        while (box < 0 && ++cw < s.bins.nw) {
            BinRange br;
            cloud_bins(s, lo3, hi3, br);
            cand = bin_candidates(s.bins, br, cw);
            box = next_box(s, lo3, hi3, cw, cand);
        }
        if (box < 0) return;
        faces = cut_faces(nom, c6, s.raw + box * 6, all_faces);
#pragma unroll
        for (int i = 0; i < W; ++i) hit[i] = 0xFFFFFFFFu;
    };
    for (;;) {
        // boxes and waypoints that are done
        bool ends = false;
        int popc = 0;
        const bool next = active && faces == 0;
        if (next) {
#pragma unroll
            for (int i = 0; i < W; ++i) acc[i] |= box >= 0 ? hit[i] : 0u;
            advance_box();
            if (box < 0) {
                popc = set_count<W>(acc);
                ends = wm == 0u || popc >= a.c_cut;
            }
        }
        n.bt += lanes_of(next && box >= 0);
        bool dominated = false;
        if (ends) {
            const int sl = mine.sl;
            bool keep = popc < a.c_cut;
            dominated = keep && a.preprune &&
                        stair_get(a.stair, a.stair_w, (int)(mine.nodes >> 16), popc) < mine.cost;
            keep &= !dominated;
            a.c_flag[sl] = keep ? 1 : 0;
            a.c_pop[sl] = popc;
            if (keep) store_set<W>(a.c_mask + (size_t)sl * W, acc);
            active = false;
        }
        n.pre += lanes_of(dominated);
        // flagged decisions of the pairs below the cut with a particle close
        // to a face, one pair at a time
        unsigned long long todo = __ballot(ends && close != 0u && popc < a.c_cut);
        while (todo) {
            const int src = __ffsll((long long)todo) - 1;
            todo &= todo - 1ull;
            const int i = (threadIdx.x & ~63) + src, from = ((l.mine[i].ks >> 8) + 1) & 31;
            const uint32_t c = (uint32_t)__shfl((int)close, src, 64);   // (by step)
            n.flag += flagged_count<N>(a, l.mine[i], l.mine_near[i], c >> from | c << ((32 - from) & 31), s);
        }
        // new records
        const unsigned long long idle = __ballot(!active);
        if (left && (int)__popcll(idle) >= kRefill) {
            int first = 0;
            if (lane == 0) first = atomicAdd(l.cnt + 2, (int)__popcll(idle));
            first = __shfl(first, 0, 64);
            left = first + (int)__popcll(idle) < n_list;
            const int i = first + (int)__popcll(idle & lanemask_lt(lane));
            if (!active && i < n_list) {
                const PairRec rec = l.list[i];
                wm = l.near[i];
                l.mine[threadIdx.x] = rec;
                l.mine_near[threadIdx.x] = wm;
                load_set<W>(a.p_mask + (size_t)rec.p * W, acc);
                active = true;
                close = 0u;
                box = -1;
            }
        }
        if (!left) {
            const int busy = lanes_of(active);
            if (busy == 0 || (more && busy < kLow)) break;
        }
        // new waypoints (a marked one meets at least one box)
        const bool move = active && box < 0;
        n.wp += lanes_of(move);
        if (move) {
            const int k = __ffs((int)wm);
            wm &= wm - 1u;
            const PairRec rec = mine;
            st = (rec.ks >> 8) + k;
            load_cloud(a.cloud + (size_t)st * 6, c6);
            {
                Cubic cs[3];
                const double dtk = record_cubics(a, rec, cs);
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) nom[ax] = cs[ax].at((double)k * dtk);
            }
            float lo3[3], hi3[3];
            cloud_box(nom, c6, lo3, hi3);
            BinRange br;
            cloud_bins(s, lo3, hi3, br);
            cw = 0;
            cand = bin_candidates(s.bins, br, 0);
            advance_box();
        }
        n.bt += lanes_of(move && box >= 0);
        // one face
        if (active && faces != 0) {
            const int f = __ffs(faces) - 1;
            faces &= faces - 1;
            bool c = false;
            face_hits<N>(a, s, nom, c6, st, box, f, hit, c);
            close |= (c ? 1u : 0u) << (st & 31);
        }
    }
    nomv = Vec4d{nom[0], nom[1], nom[2], 0.0};
    c6v = Vec8f{c6[0], c6[1], c6[2], c6[3], c6[4], c6[5], 0.0f, 0.0f};
}

// The same for a list that leaves lanes over, 2^sh lanes a record (whole
// workgroup, n_list << sh <= blockDim.x): a group's lanes take the next
// waypoints of the record side by side, and the hits are joined in waypoint
// order, so the record stops at the waypoint where test_records would (the
// waypoints past it count for nothing).  A small round's time is its longest
// record's chain of steps, which this shortens by up to 2^sh: the 2,333-sample
// query's expansion (147,743 waypoints of 42,813 pairs in seven rounds) took
// 1.16 ms a record per lane.
template <int N>
__device__ __forceinline__ void test_records_several(const RoundArgs& a, const BoxLds& s,
                                                  const PairLds& l, int n_list, int sh,
                                                  bool all_faces, PairCounts& n) {
    constexpr int W = N / 32;
    const int lane = threadIdx.x & 63, G = 1 << sh, g = lane & (G - 1);
    const int rec_i = threadIdx.x >> sh;
    bool go = rec_i < n_list;
    if (__ballot(go) == 0ull) return;
    const PairRec& rec = l.list[go ? rec_i : 0];
    uint32_t wm = go ? l.near[rec_i] : 0u;   // marked waypoints left
    uint32_t acc[W];                         // the parent's bits and the hits so far
    load_set<W>(a.p_mask + (size_t)rec.p * W, acc);
    uint32_t close_at = 0u;                  // waypoints with a particle close to a face
    while (__ballot(go) != 0ull) {
        // this lane's waypoint: the g-th marked one from here on
        uint32_t m = wm;
        for (int j = 0; j < g; ++j) m &= m - 1u;
        const int k = go ? __ffs((int)m) : 0;
        uint32_t sum[W];
#pragma unroll
        for (int i = 0; i < W; ++i) sum[i] = 0u;
        bool close = false;
        int n_bt = 0;
        if (k) {
            const int st = (rec.ks >> 8) + k;
            double nom[3];
            float c6[6], lo3[3], hi3[3];
            load_cloud(a.cloud + (size_t)st * 6, c6);
            {
                Cubic cs[3];
                const double dtk = record_cubics(a, rec, cs);
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) nom[ax] = cs[ax].at((double)k * dtk);
            }
            cloud_box(nom, c6, lo3, hi3);
            BinRange br;
            cloud_bins(s, lo3, hi3, br);
            for (int w = 0; w < s.bins.nw; ++w) {
                unsigned long long cand = bin_candidates(s.bins, br, w);
                for (int box; (box = next_box(s, lo3, hi3, w, cand)) >= 0;) {
                    ++n_bt;
                    uint32_t hit[W];
#pragma unroll
                    for (int i = 0; i < W; ++i) hit[i] = 0xFFFFFFFFu;
                    int faces = cut_faces(nom, c6, s.raw + box * 6, all_faces);
                    while (faces) {
                        const int f = __ffs(faces) - 1;
                        faces &= faces - 1;
                        face_hits<N>(a, s, nom, c6, st, box, f, hit, close);
                    }
#pragma unroll
                    for (int i = 0; i < W; ++i) sum[i] |= hit[i];
                }
            }
        }
        // hits of the group's waypoints up to each lane's
        for (int o = 1; o < G; o <<= 1) {
#pragma unroll
            for (int i = 0; i < W; ++i) {
                const uint32_t y = (uint32_t)__shfl_up((int)sum[i], o, 64);
                sum[i] |= g >= o ? y : 0u;
            }
        }
        int cnt = 0;
#pragma unroll
        for (int i = 0; i < W; ++i) cnt += __popc(sum[i] | acc[i]);
        // where the record stops: the first lane that reaches the cutoff, or
        // the last with a waypoint
        const int g0 = lane & ~(G - 1);
        const uint32_t all = G == 32 ? 0xFFFFFFFFu : (1u << G) - 1u;
        const uint32_t cut = (uint32_t)(__ballot(k && cnt >= a.c_cut) >> g0) & all;
        const uint32_t have = (uint32_t)(__ballot(k != 0) >> g0) & all;
        const int stop = cut ? __ffs((int)cut) - 1 : __popc(have) - 1;
        const bool counts = k != 0 && g <= stop;
        n.wp += lanes_of(counts);
        {
            int v = counts ? n_bt : 0;
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            n.bt += v;
        }
        if (__ballot(counts && close) != 0ull) {
            uint32_t c = counts && close ? 1u << (k - 1) : 0u;
            for (int o = 1; o < G; o <<= 1) c |= (uint32_t)__shfl_xor((int)c, o, 64);
            close_at |= c;
        }
#pragma unroll
        for (int i = 0; i < W; ++i) {
            const uint32_t y = (uint32_t)__shfl((int)sum[i], g0 + max(stop, 0), 64);
            acc[i] |= go ? y : 0u;
        }
        const bool ends = go && (cut != 0u || __popc(wm) <= G);
        for (int j = 0; j < G; ++j) wm &= wm - 1u;
        const bool lead = ends && g == 0;
        bool dominated = false;
        int popc = 0;
        if (lead) {
            popc = set_count<W>(acc);
            bool keep = popc < a.c_cut;
            dominated = keep && a.preprune &&
                        stair_get(a.stair, a.stair_w, (int)(rec.nodes >> 16), popc) < rec.cost;
            keep &= !dominated;
            a.c_flag[rec.sl] = keep ? 1 : 0;
            a.c_pop[rec.sl] = popc;
            if (keep) store_set<W>(a.c_mask + (size_t)rec.sl * W, acc);
        }
        n.pre += lanes_of(dominated);
        unsigned long long todo = __ballot(lead && close_at != 0u && popc < a.c_cut);
        while (todo) {
            const int src = __ffsll((long long)todo) - 1;
            todo &= todo - 1ull;
            const int i = ((threadIdx.x & ~63) + src) >> sh;
            n.flag += flagged_count<N>(a, l.list[i], l.near[i], (uint32_t)__shfl((int)close_at, src, 64), s);
        }
        go &= !ends;
    }
}

// One pass: pairs base + thread, those pair_front keeps onto the stack.
__device__ __forceinline__ void front_pass(const RoundArgs& a, int base, int q_end, int n_B,
                                           const PairLds& l, PairCounts& n) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int tile = base + (tid & ~63), q = base + tid;
    PairRec r;
    PairFate fate = kPairNone;
    if (tile < q_end) {   // the wave's pairs
        const int grp = wave_group_of(a.b_off, n_B, tile, q);
        if (q < q_end) fate = pair_front(a, q, grp, r);
    }
    const bool go = fate == kPairGoes;
    n.drop += lanes_of(fate == kPairDropped);
    n.pre += lanes_of(fate == kPairDominated);
    const unsigned long long m = __ballot(go);
    n.sim += (int)__popcll(m);
    int wb = 0;
    if (lane == 0 && m) wb = atomicAdd(l.cnt, (int)__popcll(m));
    wb = __shfl(wb, 0, 64);
    if (go) l.front[wb + (int)__popcll(m & lanemask_lt(lane))] = r;
}

constexpr int kWideBoxes = 3;   // (see by_particle)

// Stack entries first .. first + take - 1 (take <= blockDim.x), 2^sh lanes a
// record where there are few: their marked waypoints.  Without one the pair
// keeps its parent's bits and is settled here; the others go to the list, wide ones
// to its end (with `ranked` there are none), or with `queue` to the round's queue.
template <int N>
__device__ __forceinline__ void mark_pass(const RoundArgs& a, int first, int take, const BoxLds& s,
                                          const float* gl, const float* gh, const PairLds& l,
                                          bool queue, bool ranked) {
    constexpr int W = N / 32;
    const int T = blockDim.x, tid = threadIdx.x, lane = tid & 63;
    int sh = 0;
    while (sh < 4 && (take << (sh + 1)) <= T) ++sh;
    if ((tid & ~63) >= (take << sh)) return;   // the wave has none
    const int i = tid >> sh, g = tid & ((1 << sh) - 1);
    const bool on = i < take;
    PairRec rec;
    uint32_t near = 0u;
    int weight = 0;
    if (on) {
        rec = l.front[first + i];
        near = mark_waypoints(a, rec, s, gl, gh, 1 + g, 1 << sh, weight);
    }
    for (int o = 1; o < (1 << sh); o <<= 1) {
        near |= (uint32_t)__shfl_xor((int)near, o, 64);
        weight += __shfl_xor(weight, o, 64);
    }
    const bool lead = on && g == 0;
    if (lead && near == 0u) {
        uint32_t bits[W];
        load_set<W>(a.p_mask + (size_t)rec.p * W, bits);
        a.c_flag[rec.sl] = 1;
        a.c_pop[rec.sl] = set_count<W>(bits);
        store_set<W>(a.c_mask + (size_t)rec.sl * W, bits);
    }
    const bool test = lead && near != 0u;
    const bool wide = test && !ranked && weight >= kWideBoxes * (int)__popc(near);
    const bool front = test && !wide;
    const unsigned long long m = __ballot(front), wides = __ballot(wide);
    if (queue) {
        const unsigned long long all = m | wides;
        int at = 0;
        if (lane == 0 && all) {
            at = atomicAdd(&a.ctl->n_tasks, (int)__popcll(all));
            atomicAdd(l.cnt + 5, kWideShare * (int)__popcll(wides) - (int)__popcll(all));
        }
        at = __shfl(at, 0, 64) + (int)__popcll(all & lanemask_lt(lane));
        if (test) {
            a.c_pos[at] = rec.sl;
            a.c_pop[rec.sl] = (int32_t)near;
        }
        return;
    }
    int wb = 0;
    if (lane == 0 && m) wb = atomicAdd(l.cnt + 1, (int)__popcll(m));
    if (lane == 1 && wides) wb = atomicAdd(l.cnt + 3, (int)__popcll(wides));
    const int w0 = __shfl(wb, 0, 64), w1 = __shfl(wb, 1, 64);
    if (test) {
        const int k = wide ? T - 1 - (w1 + (int)__popcll(wides & lanemask_lt(lane)))
                           : w0 + (int)__popcll(m & lanemask_lt(lane));
        l.list[k] = rec;
        l.near[k] = near;
    }
}

// The wide records at the list's end, a wave each.
template <int N>
__device__ __forceinline__ void test_wide(const RoundArgs& a, const BoxLds& s, const PairLds& l, PairCounts& n) {
    const int n_list = l.cnt[3];
    if (n_list == 0) return;
    for (;;) {
        int i = 0;
        if ((threadIdx.x & 63) == 0) i = atomicAdd(l.cnt + 4, 1);
        i = uniform(i);
        if (i >= n_list) return;
        const int k = blockDim.x - 1 - i;
        by_particle<N>(a, s, uniform(l.list[k]), uniform(l.near[k]), n);
    }
}

// This workgroup's share (rank of `size`) of the pairs q0 .. q_end - 1.  With
// more than blockDim.x pairs a workgroup, passes of blockDim.x strided over
// the workgroups:
//   1. pair_front over passes until a full workgroup of pairs has passed it
//      (or the pairs end);
//   2. their marked waypoints, a record per thread;
//   3. the particles of those with any, a record per lane (test_records).
// With fewer, one short pass each, so that every workgroup has some (a few
// hundred pairs make a whole round of a small query), and several lanes for
// each record it gets (test_records_several).  l.cnt is zero on entry and on
// return; the counts are added to tot.  With `queue` the marked records are left to
// queued_by_particle.  With NaN deviations, whose particles only the rank tables
// leave out, every record is tested by rank.
template <int N>
__device__ __forceinline__ void expand_box_block(const RoundArgs& a, int q0, int q_end, int rank,
                                                 int size, int n_B, const BoxLds& s, const float* gl,
                                                 const float* gh, const PairLds& l, bool queue, PairTotals* tot) {
    constexpr int W = N / 32;
    constexpr int kLeast = 8;   // pairs of a short pass
    PairCounts n;
    const int T = blockDim.x, tid = threadIdx.x;
    const int per = max((q_end - q0 + size - 1) / size, kLeast);
    const bool all_faces = *a.rank_nan != 0;
    queue &= !all_faces;
    auto leave = [&]() {   // (one thread, between barriers)
        if (l.cnt[5] && !all_faces) atomicAdd(&a.ctl->wide, l.cnt[5]);
        for (int k = 0; k < kPairCounters; ++k) l.cnt[k] = 0;
    };
    if (per <= T) {
        const int base = q0 + rank * per;
        if (base >= q_end) return;
        q_end = min(q_end, base + per);
        front_pass(a, base, q_end, n_B, l, n);
        __syncthreads();
        mark_pass<N>(a, 0, l.cnt[0], s, gl, gh, l, queue, all_faces);
        __syncthreads();
        const int n_list = l.cnt[1];
        int sh = 0;
        while (sh < 4 && (n_list << (sh + 1)) <= T) ++sh;
        test_records_several<N>(a, s, l, n_list, sh, all_faces, n);
        test_wide<N>(a, s, l, n);
        add_counts(tot, n);
        __syncthreads();
        if (tid == 0) {
            if (l.cnt[3]) l.cnt[5] += (kWideShare - 1) * l.cnt[3] - l.cnt[1];
            leave();
        }
        __syncthreads();
        return;
    }
    int base = q0 + rank * T;
    const int stride = size * T;
    Vec4d nom = Vec4d{0.0, 0.0, 0.0, 0.0};
    Vec8f c6 = Vec8f{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    uint32_t acc[W], hit[W];
    unsigned long long cand = 0ull;
    uint32_t wm = 0u;
    int st = 0, box = -1, cw = 0, faces = 0;
    bool active = false;
    uint32_t close = 0u;
    int have = 0;   // stack entries (this and base are the same in every thread)
    while (base < q_end || have > 0) {
        while (have < T && base < q_end) {
            front_pass(a, base, q_end, n_B, l, n);
            __syncthreads();
            have = l.cnt[0];
            __syncthreads();   // (read everywhere before it changes)
            base += stride;
        }
        const int take = min(have, T);
        have -= take;
        mark_pass<N>(a, have, take, s, gl, gh, l, queue, all_faces);
        __syncthreads();
        test_records<N>(a, s, l, l.cnt[1], base < q_end || have > 0, all_faces, nom, c6, acc, hit,
                        cand, wm, st, box, cw, faces, active, close, n);
        test_wide<N>(a, s, l, n);
        add_counts(tot, n);
        __syncthreads();
        if (tid == 0) {
            l.cnt[0] = have;
            if (l.cnt[3]) l.cnt[5] += (kWideShare - 1) * l.cnt[3] - l.cnt[1];
            for (int k = 1; k < 5; ++k) l.cnt[k] = 0;
        }
        __syncthreads();
    }
    if (tid == 0) leave();
    __syncthreads();
}

}  // namespace pump
