// Expansion with the half-space model (Sec. III-B; the box model:
// explore_lane.hpp): pair q of group lo gets its edge and parent plan, cost,
// step count and K_e waypoints; it is dropped past S_max and resolved if the
// parent's own cp_hat already makes it dominated.  Otherwise each waypoint's
// local convex region is built plane by plane, and at those waypoints where
// some particle of the cloud's bounding box can reach a plane (or come within
// the flag distance), in their order until the pair is cut, every particle is
// tested against the planes (eq. (7)), in FP64.
//
// Two parts, with a queue between them (what stays of a group's pairs varies
// from none to all, and the second part's batches are even):
//   1. a lane per pair: header; the pairs that stay are queued;
//   2. a workgroup per batch of queued pairs: a lane per (pair, waypoint) builds
//      the region's planes, of which those within reach go to a pool in LDS,
//      chained per waypoint; then a wave per pair, particles across lanes, over
//      the chained planes.
// What bounded it was lanes without work and planes built twice: a lane per
// pair built them waypoint by waypoint up to the first within reach, and the
// particle stage, a wave per pair, built them again with a wave's reduction for
// each: 463,000 pairs over 6 rounds (4000 samples, 20 boxes, 128 particles) took
// 4.5 ms, now 0.95 (headers 0.13).
#pragma once

#include "explore_lane.hpp"
#include "explore_ops.hpp"

namespace pump {

constexpr int kHalfPairs = 32;     // most pairs of a batch
constexpr int kHalfPool = 512;     // planes in LDS (a waypoint that finds no room is rebuilt)
constexpr uint32_t kNoPlane = 0xFFFFu, kRebuild = 0xFFFEu;

struct HalfLds {
    HalfPair list[kHalfPairs];
    double plane[kHalfPool][4];                  // a, b
    double c23[kHalfPairs][6];
    float c01[kHalfPairs][6];
    uint32_t item[kHalfPairs * kMaxWaypoints];   // first plane | planes of the region << 16
    uint16_t next[kHalfPool];
    int first[kHalfPairs + 1];                   // items before the pair
    uint32_t near[kHalfPairs];
    int n_pool;
};

__host__ __device__ constexpr size_t half_lds_bytes(int n_obs) {
    return sizeof(HalfLds) + (size_t)n_obs * 6 * sizeof(double);
}

struct HalfStage {
    HalfLds* l;
    const double* boxes;
};

__device__ __forceinline__ HalfStage stage_half_lds(const RoundArgs& a, char* mem) {
    HalfStage s;
    s.l = reinterpret_cast<HalfLds*>(mem);
    double* b = reinterpret_cast<double*>(mem + sizeof(HalfLds));
    for (int t = threadIdx.x; t < a.n_obs * 6; t += blockDim.x) b[t] = (double)a.obs[t];
    s.boxes = b;
    return s;
}

// Of pair q: 0 if it is resolved, 1 if its particles matter (h: its record).
__device__ __forceinline__ int half_header(const RoundArgs& a, int q, int lo, int& n_pre, int& n_drop,
                                           HalfPair& h) {
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
        ++n_drop;
        return 0;
    }
    if (a.preprune && stair_get(a.stair, a.stair_w, x, a.p_pop[p]) < cost) {
        a.c_flag[sl] = 0;
        a.c_pop[sl] = -1;
        ++n_pre;
        return 0;
    }
    a.c_edge[sl] = e;
    a.c_cost[sl] = cost;
    a.c_step[sl] = s_p + K;
    h = HalfPair{tau, sl, p, (uint32_t)head | (uint32_t)x << 16, K, s_p};
    return 1;
}

// The nominal position and velocity at waypoint k of the pair in slot i.  At a
// node at rest the velocity is zero but for its rounding, whose direction
// decides the plane that eq. (7) leaves: its form is written out.
__device__ __forceinline__ void half_waypoint(const HalfLds& l, int i, double tau, int K, int k, double* y,
                                              double* v) {
    const double t = ((double)k * tau) / (double)K;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const Cubic c{(double)l.c01[i][2 * ax], (double)l.c01[i][2 * ax + 1], l.c23[i][2 * ax],
                      l.c23[i][2 * ax + 1]};
        y[ax] = c.at(t);
        v[ax] = fma(t, fma(t * 3.0, c.c3, 2.0 * c.c2), c.c1);
    }
}

// The planes of item j of `total` (a wave's lanes together; j >= total: no item).
__device__ __forceinline__ void half_planes(const RoundArgs& a, const HalfStage& s, int n_pairs, int j,
                                            int total) {
    HalfLds& l = *s.l;
    const int nw = (a.n_obs + 63) >> 6;
    unsigned long long rem[kMaxObsWords];
    double y[3] = {0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0};
    float cl[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    int i = 0, k = 0;
    bool on = j < total;
    for (int w = 0; w < kMaxObsWords; ++w) rem[w] = 0ull;
    if (on) {
        int hi = n_pairs;   // first[i] <= j < first[hi]
        while (hi - i > 1) {
            const int mid = (i + hi) >> 1;
            if (l.first[mid] <= j) i = mid; else hi = mid;
        }
        const HalfPair& h = l.list[i];
        k = j - l.first[i] + 1;
        half_waypoint(l, i, h.tau, h.K, k, y, v);
        const float* c = a.cloud + (size_t)(h.s_p + k) * 6;
        for (int u = 0; u < 6; ++u) cl[u] = c[u];
        all_boxes(a.n_obs, rem);
    }
    uint32_t first = kNoPlane;
    int planes = 0;
    bool near = false;
    while (__ballot(on) != 0ull) {
        double d[3], av[3], b;
        const bool found = hs_next_lanes(y, s.boxes, nw, rem, d);
        on = on && found;
        if (on) {
            ++planes;
            hs_project(d, v, av, b);
            double reach = 0.0;
            for (int ax = 0; ax < 3; ++ax)
                reach += fmax(av[ax] * (double)cl[ax], av[ax] * (double)cl[3 + ax]);
            const double na = sqrt(b), least = b - kFlagEps * na - 1e-12 * (b + 1.0);
            // (a plane at a right angle to an axis on which the cloud has no
            // bounds has no reach, 0 times infinity: it marks no waypoint, but at
            // a marked one the particles are tested against it)
            near |= reach > least;
            if (!(reach <= least)) {
                if (na > 0.0 && first != kRebuild) {
                    const int at = atomicAdd(&l.n_pool, 1);
                    if (at < kHalfPool) {
                        for (int ax = 0; ax < 3; ++ax) l.plane[at][ax] = av[ax];
                        l.plane[at][3] = b;
                        l.next[at] = (uint16_t)first;
                        first = (uint32_t)at;
                    } else {
                        first = kRebuild;
                    }
                }
            }
        }
    }
    if (j < total) {
        l.item[j] = first | (uint32_t)planes << 16;
        if (near) atomicOr(&l.near[i], 1u << (k - 1));
    }
}

// The particles of the pair in slot i, some of whose waypoints are near (whole
// wave).
// Lane l holds particles l, l + 64, ..., so the hit bits of particle row r are
// one ballot (mask words 2r and 2r+1 as they stand).  Counters are
// wave-uniform (wp: waypoints tested, bt: waypoint-plane tests).
template <int N>
__device__ __forceinline__ void half_particles(const RoundArgs& a, const HalfStage& s, int i, PairCounts& n) {
    constexpr int W = N / 32;                      // u32 mask words
    constexpr int PPL = N >= 64 ? N / 64 : 1;      // particles per lane
    HalfLds& l = *s.l;
    const int lane = threadIdx.x & 63;
    const bool valid_lane = (N >= 64) || (lane < N);
    const HalfPair h = l.list[i];
    const double cost = a.c_cost[h.sl];
    bool hit[PPL], deep[PPL], nearp[PPL], par[PPL];
    float dn[PPL][3];   // the next waypoint's deviations, asked for ahead
    auto ask = [&](int k) {
#pragma unroll
        for (int r = 0; r < PPL; ++r)
#pragma unroll
            for (int ax = 0; ax < 3; ++ax)
                dn[r][ax] = a.D[((size_t)(h.s_p + k) * 3 + ax) * N + (valid_lane ? r * 64 + lane : 0)];
    };
    unsigned wm = (unsigned)__builtin_amdgcn_readfirstlane((int)l.near[i]);
    ask(__ffs((int)wm));
#pragma unroll
    for (int r = 0; r < PPL; ++r) {
        hit[r] = deep[r] = nearp[r] = false;
        // the parent's bit of each of this lane's particles (r * 64 + lane)
        const int j = valid_lane ? r * 64 + lane : 0;
        par[r] = valid_lane && ((a.p_mask[(size_t)h.p * W + (j >> 5)] >> (j & 31)) & 1u);
    }
    // the pair stops at the waypoint where its count reaches c_cut
    while (wm) {
        ++n.wp;   // waypoints at which a plane can be reached
        const int k = __ffs((int)wm);
        wm &= wm - 1u;
        double dy[PPL][3];
#pragma unroll
        for (int r = 0; r < PPL; ++r)
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) dy[r][ax] = (double)dn[r][ax];
        if (wm) ask(__ffs((int)wm));
        auto test = [&](const double* av, double b) {
            const double na = sqrt(b);
#pragma unroll
            for (int r = 0; r < PPL; ++r) {
                const double g = (av[0] * dy[r][0] + av[1] * dy[r][1]) + av[2] * dy[r][2];
                const double mg = (g - b) / na;
                if (g > b) hit[r] = true;
                if (mg >= kFlagEps) deep[r] = true;
                if (fabs(mg) < kFlagEps) nearp[r] = true;
            }
        };
        const uint32_t it = (uint32_t)__builtin_amdgcn_readfirstlane((int)l.item[l.first[i] + k - 1]);
        n.bt += (int)(it >> 16);
        uint32_t at = it & 0xFFFFu;
        if (at == kRebuild) {   // (the pool was full)
            double y[3], v[3], d[3];
            half_waypoint(l, i, h.tau, h.K, k, y, v);
            unsigned long long rem[kMaxObsWords];
            all_boxes(a.n_obs, rem);
            while (hs_next_wave(y, s.boxes, a.n_obs, rem, d)) {
                double av[3], b;
                hs_project(d, v, av, b);
                if (sqrt(b) > 0.0) test(av, b);
            }
        } else {
            while (at != kNoPlane) {
                test(l.plane[at], l.plane[at][3]);
                at = (uint32_t)__builtin_amdgcn_readfirstlane((int)l.next[at]);
            }
        }
        int cnt = 0;
#pragma unroll
        for (int r = 0; r < PPL; ++r) cnt += (int)__popcll(__ballot(valid_lane && (hit[r] || par[r])));
        if (cnt >= a.c_cut) break;
    }
    // gather hits into the N-bit mask and OR with the parent's bits
    uint32_t words[W];
    int popc = 0, flg = 0;
#pragma unroll
    for (int r = 0; r < PPL; ++r) {
        const unsigned long long pb = __ballot(par[r]);
        const unsigned long long hb = __ballot(hit[r] && valid_lane) | pb;
        flg += (int)__popcll(__ballot(nearp[r] && !deep[r] && valid_lane) & ~pb);
        popc += (int)__popcll(hb);
        if (N >= 64) {
            words[2 * r] = (uint32_t)hb;
            words[(2 * r + 1) % W] = (uint32_t)(hb >> 32);
        } else {
            words[0] = (uint32_t)hb;
        }
    }
    bool keep = popc < a.c_cut;
    if (keep && a.preprune && stair_get(a.stair, a.stair_w, (int)(h.nodes >> 16), popc) < cost) {
        keep = false;
        ++n.pre;
    }
    if (lane == 0) {
        a.c_flag[h.sl] = keep ? 1 : 0;
        a.c_pop[h.sl] = popc;
    }
    if (keep && lane < W) {
        uint32_t v = 0;
#pragma unroll
        for (int w = 0; w < W; ++w)
            if (w == lane) v = words[w];
        a.c_mask[(size_t)h.sl * W + lane] = v;
    }
    if (popc < a.c_cut) n.flag += flg;   // flagged decisions of pairs below the cut
}

// 1. for pairs [q0, q_end) of the round: the workgroup's passes, strided over G.
__device__ __forceinline__ void half_headers(const RoundArgs& a, int q0, int q_end, int b, int G, int n_B,
                                             PairTotals* tot) {
    PairCounts n;
    const int tid = threadIdx.x, lane = tid & 63, T = blockDim.x;
    for (int base = q0 + b * T; base < q_end; base += G * T) {
        const int tile = base + (tid & ~63), q = base + tid;
        if (tile >= q_end) break;   // (whole waves)
        const int grp = wave_group_of(a.b_off, n_B, tile, q);
        HalfPair h;
        int pre = 0, drop = 0;
        const bool go = q < q_end && half_header(a, q, grp, pre, drop, h) != 0;
        n.pre += lanes_of(pre != 0);
        n.drop += lanes_of(drop != 0);
        n.sim += lanes_of(go);
        const unsigned long long m = __ballot(go);
        int at = 0;
        if (lane == 0 && m) at = atomicAdd(&a.ctl->n_tasks, (int)__popcll(m));
        at = __shfl(at, 0, 64) + (int)__popcll(m & lanemask_lt(lane));
        if (go) a.tasks[at] = h;
        add_counts(tot, n);
    }
}

// 2. for the n_tasks queued pairs: batches shared by G workgroups; all threads
// of the workgroup call it.
template <int N>
__device__ __forceinline__ void half_batches(const RoundArgs& a, int n_tasks, int b, int G, const HalfStage& s,
                                             PairTotals* tot) {
    constexpr int W = N / 32;
    PairCounts n;
    HalfLds& l = *s.l;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, T = blockDim.x;
    // pairs enough for every workgroup, else fewer of them each; some ten
    // waypoints each fill a workgroup's lanes
    const int batch = min(kHalfPairs, max(T / 64, (n_tasks + G - 1) / G));
    for (int base = b * batch; base < n_tasks; base += G * batch) {
        const int np = min(batch, n_tasks - base);
        if (wave == 0) {
            int K = 0;
            if (lane < np) {
                const HalfPair h = a.tasks[base + lane];
                l.list[lane] = h;
                K = h.K;
                Cubic cs[3];
                hermite(a.X + (size_t)(h.nodes & 0xFFFFu) * 6, a.X + (size_t)(h.nodes >> 16) * 6, h.tau, cs);
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) {
                    l.c01[lane][2 * ax] = (float)cs[ax].c0;
                    l.c01[lane][2 * ax + 1] = (float)cs[ax].c1;
                    l.c23[lane][2 * ax] = cs[ax].c2;
                    l.c23[lane][2 * ax + 1] = cs[ax].c3;
                }
            }
            int x = K;   // items up to this lane's pair
            for (int o = 1; o < 64; o <<= 1) {
                const int u = __shfl_up(x, o, 64);
                if (lane >= o) x += u;
            }
            if (lane < np) {
                l.first[lane + 1] = x;
                l.near[lane] = 0u;
            }
            if (lane == 0) {
                l.first[0] = 0;
                l.n_pool = 0;
            }
        }
        __syncthreads();
        const int total = l.first[np];
        for (int j0 = tid & ~63; j0 < total; j0 += T) half_planes(a, s, np, j0 + lane, total);
        __syncthreads();
        // pairs that keep their parent's bits
        if (tid < np && l.near[tid] == 0u) {
            const HalfPair& h = l.list[tid];
            a.c_flag[h.sl] = 1;
            a.c_pop[h.sl] = a.p_pop[h.p];
            for (int w = 0; w < W; ++w) a.c_mask[(size_t)h.sl * W + w] = a.p_mask[(size_t)h.p * W + w];
        }
        for (int i = wave; i < np; i += T >> 6)
            if (l.near[i] != 0u) half_particles<N>(a, s, i, n);
        add_counts(tot, n);
        __syncthreads();
    }
}

}  // namespace pump
