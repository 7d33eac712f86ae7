// Explore (Alg. 4): one round = expand the group B to every neighbour,
// RemoveDominated, retire B, select the next group.
#include <algorithm>

#include "explore_half.hpp"
#include "explore_lane.hpp"

namespace pump {

// ---------------------------------------------------------------------------
// Device-wide exclusive scan of int32 (length read from device memory).
// ---------------------------------------------------------------------------
__device__ __forceinline__ int block_exclusive_sum(int v, int* s_tmp, int& total) {
    // 256 threads = 4 waves
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) s_tmp[wave] = x;
    __syncthreads();
    int off = 0;
    for (int w = 0; w < wave; ++w) off += s_tmp[w];
    total = s_tmp[0] + s_tmp[1] + s_tmp[2] + s_tmp[3];
    __syncthreads();
    return off + x - v;
}

// One or two arrays (grid.y) per launch.
__global__ __launch_bounds__(256) void k_scan_reduce(ScanJob j0, ScanJob j1) {
    __shared__ int s_tmp[4];
    const ScanJob& j = blockIdx.y ? j1 : j0;
    const int n = *j.n;
    const int base = blockIdx.x * kScanBlock;
    if (base >= n) {
        if (threadIdx.x == 0) j.blk[blockIdx.x] = 0;
        return;
    }
    int sum = 0;
    for (int k = 0; k < 4; ++k) {
        int idx = base + threadIdx.x * 4 + k;
        if (idx < n) sum += j.in[idx];
    }
    int total;
    block_exclusive_sum(sum, s_tmp, total);
    if (threadIdx.x == 0) j.blk[blockIdx.x] = total;
}

// Block totals to their exclusive sums (one workgroup an array).
__global__ __launch_bounds__(256) void k_scan_blocks(ScanJob j0, ScanJob j1, int nblk) {
    __shared__ int s_tmp[4];
    const ScanJob& j = blockIdx.y ? j1 : j0;
    int carry = 0;
    for (int b0 = 0; b0 < nblk; b0 += 256) {
        int idx = b0 + threadIdx.x;
        int v = idx < nblk ? j.blk[idx] : 0;
        int total;
        int ex = block_exclusive_sum(v, s_tmp, total);
        if (idx < nblk) j.blk[idx] = carry + ex;
        carry += total;
    }
}

// summed: blk holds exclusive sums, else totals, which every workgroup adds up
// to its own place.  The last workgroup writes the array's total.
__global__ __launch_bounds__(256) void k_scan_down(ScanJob j0, ScanJob j1, int summed) {
    __shared__ int s_tmp[4];
    const ScanJob& j = blockIdx.y ? j1 : j0;
    const int n = *j.n;
    const int base = blockIdx.x * kScanBlock;
    const bool last = blockIdx.x == gridDim.x - 1;
    if (base >= n && !last) return;
    int before = 0;
    if (summed) {
        before = j.blk[blockIdx.x];
    } else {
        for (int k = threadIdx.x; k < (int)blockIdx.x; k += 256) before += j.blk[k];
        int total;
        block_exclusive_sum(before, s_tmp, total);
        before = total;
    }
    int v[4];
    int sum = 0;
    for (int k = 0; k < 4; ++k) {
        int idx = base + threadIdx.x * 4 + k;
        v[k] = idx < n ? j.in[idx] : 0;
        sum += v[k];
    }
    int total;
    int ex = block_exclusive_sum(sum, s_tmp, total) + before;
    for (int k = 0; k < 4; ++k) {
        int idx = base + threadIdx.x * 4 + k;
        if (idx < n) j.out[idx] = ex;
        ex += v[k];
    }
    if (last && threadIdx.x == 0) {
        *j.total = before + total;
        if (j.total2) *j.total2 = before + total;
    }
}

// Each of these kernels takes some 4 us whatever it does, so two arrays of a
// step share their launches, and up to kScanDirect workgroups add up the totals
// before them by themselves (a launch less; at 1,250 of them, the indoor
// query's rounds, 4.4 us against 4.3 + 5.4).  Beyond, those reads would grow
// with the square of the length.
constexpr int kScanDirect = 2048;

void scan_exclusive2(hipStream_t s, const ScanJob& j0, const ScanJob* j1, int32_t n_upper) {
    int nblk = (n_upper + kScanBlock - 1) / kScanBlock;
    if (nblk < 1) nblk = 1;
    const dim3 grid(nblk, j1 ? 2 : 1);
    const ScanJob b = j1 ? *j1 : j0;
    k_scan_reduce<<<grid, 256, 0, s>>>(j0, b);
    const bool summed = nblk > kScanDirect;
    if (summed) k_scan_blocks<<<dim3(1, grid.y), 256, 0, s>>>(j0, b, nblk);
    k_scan_down<<<grid, 256, 0, s>>>(j0, b, summed ? 1 : 0);
}

void scan_exclusive(hipStream_t s, const int32_t* in, int32_t* out, const int32_t* n_dev,
                    int32_t n_upper, int32_t* total_dev, int32_t* blk, int32_t* total2_dev) {
    scan_exclusive2(s, ScanJob{in, out, n_dev, total_dev, total2_dev, blk}, nullptr, n_upper);
}

// ---------------------------------------------------------------------------
// Initialisation (Alg. 4 first lines): P_open = P(x_init) = B = {root},
// root = (x_init, [], 0, 0), i = 0.  The dominance staircase of every node
// starts empty (+inf); the root puts cost 0 at every pop level of node 0.
// ---------------------------------------------------------------------------
__global__ void k_init_fill(RoundArgs a, int n_nodes, unsigned* zero, int n_zero) {
    const size_t t0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    explore_init_fill(a, n_nodes, t0, stride);
    for (size_t t = t0; t < (size_t)n_zero; t += stride) zero[t] = 0u;
}

// The whole control block is cleared before the root's fields are set.
__global__ void k_root(RoundArgs a, int N) {
    unsigned* w = reinterpret_cast<unsigned*>(a.ctl);
    for (int t = threadIdx.x; t < (int)(sizeof(Ctl) / sizeof(unsigned)); t += blockDim.x) w[t] = 0u;
    __syncthreads();
    if (threadIdx.x == 0 && blockIdx.x == 0) explore_init_root(a, N);
}

void launch_explore_init(hipStream_t s, const RoundArgs& a, int n_nodes, int N, unsigned* zero,
                         int n_zero) {
    size_t n = (size_t)n_nodes * a.stair_w;
    if ((size_t)n_zero > n) n = (size_t)n_zero;
    size_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    k_init_fill<<<(unsigned)blocks, 256, 0, s>>>(a, n_nodes, zero, n_zero);
    k_root<<<1, 64, 0, s>>>(a, N);
}

// ---------------------------------------------------------------------------
// Counter partials: each workgroup adds its sums to its own slots of a.part
// (no atomics on the control block, whose one line every workgroup would
// otherwise queue on); k_counters_reduce folds them in once a round.
// ---------------------------------------------------------------------------
// Sum over the workgroup, valid in thread 0 (all threads call it; s holds
// blockDim.x / 64 entries).
__device__ __forceinline__ long long block_sum(long long v, long long* s) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    long long t = 0;
    if (threadIdx.x == 0)
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += s[w];
    __syncthreads();
    return t;
}

__device__ __forceinline__ void part_add(const RoundArgs& a, int k, long long v) {
    if (v) a.part[(size_t)blockIdx.x * kPartK + k] += v;   // this workgroup's slot
}

// kReduceBlocks workgroups, each over its share of the slots; each adds its
// sums into the control block (a handful of atomics in all).
constexpr int kReduceBlocks = 16;

__global__ __launch_bounds__(256) void k_counters_reduce(RoundArgs a, int add) {
    __shared__ long long s[4];
    long long v[kPartK];
    for (int k = 0; k < kPartK; ++k) v[k] = 0;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < kPartSlots; t += gridDim.x * blockDim.x) {
        for (int k = 0; k < kPartK; ++k) {
            v[k] += a.part[(size_t)t * kPartK + k];
            a.part[(size_t)t * kPartK + k] = 0;
        }
    }
    long long tot[kPartK];
    for (int k = 0; k < kPartK; ++k) tot[k] = block_sum(v[k], s);
    if (threadIdx.x == 0 && add) {
        Ctl* c = a.ctl;
        auto add_ll = [](long long* dst, long long x) {
            if (x) atomicAdd((unsigned long long*)dst, (unsigned long long)x);
        };
        add_ll(&c->simulated, tot[kPartSimulated]);
        add_ll(&c->preprune, tot[kPartPreprune]);
        add_ll(&c->dropped_steps, tot[kPartDropped]);
        add_ll(&c->flagged, tot[kPartFlagged]);
        add_ll(&c->sim_waypoints, tot[kPartWaypoints]);
        add_ll(&c->sim_box_tests, tot[kPartBoxTests]);
        add_ll(&c->inserted, tot[kPartInserted]);
    }
}

void launch_counters_reduce(hipStream_t s, const RoundArgs& a) {
    k_counters_reduce<<<kReduceBlocks, 256, 0, s>>>(a, 1);
}

void launch_counters_clear(hipStream_t s, const RoundArgs& a) {
    k_counters_reduce<<<kReduceBlocks, 256, 0, s>>>(a, 0);
}

// workgroups of k_expand_box: three per CU, what fits at once, so that each
// takes many passes and drains its last records only once
constexpr int kBoxGrid = 768;

static int part_grid(long long n, int per_block) {
    long long b = (n + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > kPartSlots) b = kPartSlots;
    return (int)b;
}

// ---------------------------------------------------------------------------
// Expansion (Alg. 4: every pair (p in B, x in N(p.head)) forms q with
// Cost and CP_hat, then the CP cutoff): explore_lane.hpp (box model),
// explore_half.hpp (half-space model).
// ---------------------------------------------------------------------------
// The workgroup's totals to its counter slots (after all of its waves' counts).
__device__ __forceinline__ void expand_counts(const RoundArgs& a, const PairTotals& tot) {
    __syncthreads();
    if (threadIdx.x == 0 && !a.quiet) {
        part_add(a, kPartSimulated, (long long)tot.sim);
        part_add(a, kPartPreprune, (long long)tot.pre);
        part_add(a, kPartDropped, (long long)tot.drop);
        part_add(a, kPartFlagged, (long long)tot.flag);
        part_add(a, kPartWaypoints, (long long)tot.wp);
        part_add(a, kPartBoxTests, (long long)tot.bt);
    }
}

template <int N>
__global__ __launch_bounds__(256, 3) void k_expand_box(RoundArgs a) {
    extern __shared__ __align__(16) char s_box[];
    __shared__ __align__(16) char s_pair[pair_lds_bytes(256)];
    __shared__ PairTotals s_tot;
    const BoxLds box = stage_box_lds(a, s_box);
    const PairLds pl = pair_lds(s_pair, 256);
    if (threadIdx.x < kPairCounters) pl.cnt[threadIdx.x] = 0;
    if (threadIdx.x == 0) s_tot = PairTotals{};
    __syncthreads();
    // pairs [a.q0, q_end) of the round: all of them, or one chunk
    const int q_end = a.chunked ? a.q0 + a.ctl->chunk_n : a.ctl->n_pairs;
    float gl[3], gh[3];
    for (int k = 0; k < 3; ++k) { gl[k] = a.gcloud[k]; gh[k] = a.gcloud[3 + k]; }
    expand_box_block<N>(a, a.q0, q_end, blockIdx.x, gridDim.x, a.ctl->n_B, box, gl, gh, pl, a.queue != 0,
                        &s_tot);
    expand_counts(a, s_tot);
}

template <int N>
__global__ __launch_bounds__(256, 4) void k_by_particle(RoundArgs a) {
    extern __shared__ __align__(16) char s_box[];
    __shared__ PairTotals s_tot;
    const int n_tasks = a.ctl->n_tasks;
    if ((int)blockIdx.x * 4 >= n_tasks) return;
    const BoxLds box = stage_box_lds(a, s_box);
    if (threadIdx.x == 0) s_tot = PairTotals{};
    __syncthreads();
    queued_by_particle<N>(a, n_tasks, blockIdx.x, gridDim.x, box, &s_tot);
    expand_counts(a, s_tot);
}

__global__ __launch_bounds__(256) void k_half_headers(RoundArgs a) {
    __shared__ PairTotals s_tot;
    if (threadIdx.x == 0) s_tot = PairTotals{};
    __syncthreads();
    // pairs [a.q0, q_end) of the round: all of them, or one chunk
    const int q_end = a.chunked ? a.q0 + a.ctl->chunk_n : a.ctl->n_pairs;
    half_headers(a, a.q0, q_end, blockIdx.x, gridDim.x, a.ctl->n_B, &s_tot);
    expand_counts(a, s_tot);
}

template <int N>
__global__ __launch_bounds__(256, N == 256 ? 3 : 4) void k_half_batches(RoundArgs a) {
    extern __shared__ __align__(16) char s_half[];
    __shared__ PairTotals s_tot;
    const int n_tasks = a.ctl->n_tasks;
    if ((int)blockIdx.x * 4 >= n_tasks) return;   // (a batch is at least 4 pairs)
    const HalfStage half = stage_half_lds(a, s_half);
    if (threadIdx.x == 0) s_tot = PairTotals{};
    __syncthreads();
    half_batches<N>(a, n_tasks, blockIdx.x, gridDim.x, half, &s_tot);
    expand_counts(a, s_tot);
}

// Workgroups of the second part: as many as the CUs hold at once, so that its
// batches are even (a workgroup per 32 pairs with their headers: 1.34 ms
// instead of 0.95 on the case above; 768 workgroups, some 100 pairs each: 1.75).
constexpr int kHalfGrid = 1024;
constexpr int kParticleGrid = 1024;   // likewise of the queued records

// part 1: the half-space model's headers; part 2: the rest (all of the box
// model's expansion).
template <int N>
static void launch_expand_n(hipStream_t s, const RoundArgs& a, int32_t n_pairs, int part) {
    if (a.cp_model == 0) {
        if (part & 2) {
            k_expand_box<N><<<(unsigned)std::min(part_grid(n_pairs, 16), kBoxGrid), 256,
                              box_lds_bytes(a.n_obs), s>>>(a);
            if (a.queue)
                k_by_particle<N><<<kParticleGrid, 256, box_lds_bytes(a.n_obs), s>>>(a);
        }
        return;
    }
    if (part & 1) k_half_headers<<<part_grid(n_pairs, 256), 256, 0, s>>>(a);
    if (part & 2)
        k_half_batches<N><<<(unsigned)std::min(part_grid(n_pairs, 4), kHalfGrid), 256, half_lds_bytes(a.n_obs),
                            s>>>(a);
}

void launch_expand(hipStream_t s, const RoundArgs& a, int N, int32_t n_pairs, int part) {
    if (n_pairs <= 0) return;
    switch (N) {
        case 32: launch_expand_n<32>(s, a, n_pairs, part); break;
        case 64: launch_expand_n<64>(s, a, n_pairs, part); break;
        case 128: launch_expand_n<128>(s, a, n_pairs, part); break;
        default: launch_expand_n<256>(s, a, n_pairs, part); break;
    }
}

// RemoveDominated (staircase update, then marks; see explore_ops.hpp).
__global__ __launch_bounds__(256) void k_stair_update(RoundArgs a) {
    const int n_pairs = a.chunked ? a.ctl->chunk_n : a.ctl->n_pairs;
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < n_pairs; q += gridDim.x * blockDim.x)
        stair_update_pair(a, q);
}

__global__ __launch_bounds__(256) void k_mark(RoundArgs a) {
    __shared__ long long s_ll[4];
    const int n_pairs = a.ctl->n_pairs;
    const int n_open = a.ctl->n_open;
    const int total = n_pairs + n_open;
    long long kept = 0;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < total; t += gridDim.x * blockDim.x) {
        if (t < n_pairs) kept += mark_pair(a, t) ? 1 : 0;
        else mark_open(a, t - n_pairs);
    }
    const long long t_kept = block_sum(kept, s_ll);
    if (threadIdx.x == 0) part_add(a, kPartInserted, t_kept);
}

static int grid_of(long long n) {
    long long b = (n + 255) / 256;
    if (b < 1) b = 1;
    if (b > 16384) b = 16384;
    return (int)b;
}

void launch_prune(hipStream_t s, const RoundArgs& a, int N, int32_t n_pairs, int32_t n_open) {
    (void)N;
    int b1 = (n_pairs + 255) / 256;
    if (b1 < 1) b1 = 1;
    if (b1 > 16384) b1 = 16384;
    k_stair_update<<<b1, 256, 0, s>>>(a);
    k_mark<<<part_grid((long long)n_pairs + n_open, 256), 256, 0, s>>>(a);
}

// Compaction: P_open <- (P_open \ B \ removed) U survivors.
// scan_total[0] = survivors, scan_total[1] = open plans kept.
template <int W>
__global__ __launch_bounds__(256) void k_compact(RoundArgs a) {
    const int n_pairs = a.ctl->n_pairs;
    const int n_open = a.ctl->n_open;
    const int n_plans = a.ctl->n_plans;
    const int n_surv = a.ctl->scan_total[0];
    const int n_keep = a.ctl->scan_total[1];
    const bool fits = (long long)n_plans + n_surv <= a.cap_plans;
    const int i_round = a.ctl->i;
    const int total = n_pairs + n_open;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < total; t += gridDim.x * blockDim.x) {
        if (t < n_pairs) {
            if (fits) compact_pair<W>(a, t, n_plans, n_keep, i_round);
        } else {
            compact_open(a, t - n_pairs);
        }
    }
}

__global__ void k_compact_finalize(Ctl* c, int64_t cap) { compact_finalize(c, cap); }

void launch_compact(hipStream_t s, const RoundArgs& a, int N, int32_t n_pairs, int32_t n_open,
                    int32_t* blk) {
    const ScanJob opens{a.o_keep, a.o_keep, &a.ctl->n_open, &a.ctl->scan_total[1], nullptr, blk + 65536};
    scan_exclusive2(s, ScanJob{a.c_pos, a.c_pos, &a.ctl->n_pairs, &a.ctl->scan_total[0], nullptr, blk}, &opens,
                    n_pairs > n_open ? n_pairs : n_open);
    int b = (n_pairs + n_open + 255) / 256;
    if (b < 1) b = 1;
    if (b > 16384) b = 16384;
    switch (N / 32) {
        case 1: k_compact<1><<<b, 256, 0, s>>>(a); break;
        case 2: k_compact<2><<<b, 256, 0, s>>>(a); break;
        case 4: k_compact<4><<<b, 256, 0, s>>>(a); break;
        default: k_compact<8><<<b, 256, 0, s>>>(a); break;
    }
    k_compact_finalize<<<1, 1, 0, s>>>(a.ctl, a.cap_plans);
}

// ---------------------------------------------------------------------------
// A round with more pairs than candidate slots runs in chunks of the pair
// list, in two passes.  RemoveDominated's outcome depends only on the final
// staircase of each node (the minimum over every kept candidate of the round
// and the plans before it), so
//   pass 1: per chunk, expansion and the staircase update (the candidates
//           are then dropped);
//   then:   the open list is marked against the final staircase and
//           compacted (P_open \ B \ removed);
//   pass 2: per chunk, the expansion again (the same candidates), marks
//           against the final staircase and compaction of the survivors
//           after those of the chunks before it.
// Survivors get the plan ids and open-list places the round would give them
// in one piece (pair order).  A pass-1 expansion already sees the entries of
// earlier chunks, so it may resolve a pair without simulating it that the
// round in one piece would simulate and then remove: that pair is dominated
// either way, and the staircase it would have updated already holds a lower
// cost at every level it reaches.  The counters count pass 1 (and the
// candidates kept before the test in pass 2).
// ---------------------------------------------------------------------------
__global__ void k_chunk_begin(Ctl* c, int32_t n) {
    c->chunk_n = n;
    c->n_tasks = 0;
    c->wide = 0;
}

__global__ __launch_bounds__(256) void k_mark_open_only(RoundArgs a) {
    const int n_open = a.ctl->n_open;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_open; i += gridDim.x * blockDim.x)
        mark_open(a, i);
}

__global__ __launch_bounds__(256) void k_compact_open_only(RoundArgs a) {
    const int n_open = a.ctl->n_open;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_open; i += gridDim.x * blockDim.x)
        compact_open(a, i);
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctl->chunk_base = 0;
}

__global__ __launch_bounds__(256) void k_mark_chunk(RoundArgs a) {
    __shared__ long long s_ll[4];
    const int n = a.ctl->chunk_n;
    long long kept = 0;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x)
        kept += mark_pair(a, t) ? 1 : 0;
    const long long t_kept = block_sum(kept, s_ll);
    if (threadIdx.x == 0) part_add(a, kPartInserted, t_kept);
}

// survivors of this chunk after those of the chunks before it; nothing is
// written once the plan store would overflow (the final check reports it)
template <int W>
__global__ __launch_bounds__(256) void k_compact_chunk(RoundArgs a) {
    const int n = a.ctl->chunk_n;
    const int base = a.ctl->chunk_base;
    const int n_plans = a.ctl->n_plans;
    const int n_keep = a.ctl->scan_total[1];
    const bool fits = (long long)n_plans + base + a.ctl->scan_total[0] <= a.cap_plans;
    if (!fits) return;
    const int i_round = a.ctl->i;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x)
        compact_pair<W>(a, t, n_plans + base, n_keep + base, i_round);
}

__global__ void k_chunk_end(Ctl* c) { c->chunk_base += c->scan_total[0]; }

__global__ void k_chunks_finalize(Ctl* c, int64_t cap) {
    c->scan_total[0] = c->chunk_base;
    compact_finalize(c, cap);
}

void launch_chunk_begin(hipStream_t s, const RoundArgs& a, int32_t n) {
    k_chunk_begin<<<1, 1, 0, s>>>(a.ctl, n);
}

void launch_stair_update(hipStream_t s, const RoundArgs& a, int32_t n) {
    k_stair_update<<<grid_of(n), 256, 0, s>>>(a);
}

void launch_open_compact(hipStream_t s, const RoundArgs& a, int32_t n_open, int32_t* blk) {
    k_mark_open_only<<<grid_of(n_open), 256, 0, s>>>(a);
    scan_exclusive(s, a.o_keep, a.o_keep, &a.ctl->n_open, n_open, &a.ctl->scan_total[1],
                   blk + 65536);
    k_compact_open_only<<<grid_of(n_open), 256, 0, s>>>(a);
}

void launch_chunk_compact(hipStream_t s, const RoundArgs& a, int N, int32_t n, int32_t* blk) {
    k_mark_chunk<<<part_grid(n, 256), 256, 0, s>>>(a);
    scan_exclusive(s, a.c_pos, a.c_pos, &a.ctl->chunk_n, n, &a.ctl->scan_total[0], blk);
    switch (N / 32) {
        case 1: k_compact_chunk<1><<<grid_of(n), 256, 0, s>>>(a); break;
        case 2: k_compact_chunk<2><<<grid_of(n), 256, 0, s>>>(a); break;
        case 4: k_compact_chunk<4><<<grid_of(n), 256, 0, s>>>(a); break;
        default: k_compact_chunk<8><<<grid_of(n), 256, 0, s>>>(a); break;
    }
    k_chunk_end<<<1, 1, 0, s>>>(a.ctl);
}

void launch_chunks_finalize(hipStream_t s, const RoundArgs& a) {
    k_chunks_finalize<<<1, 1, 0, s>>>(a.ctl, a.cap_plans);
}

// Next group (Alg. 4: i <- i + 1, B <- cheap open plans) and the loop test.
__global__ __launch_bounds__(256) void k_open_min(RoundArgs a) {
    // after a failed compaction (plan store full: err set, done set) the
    // open list holds only the kept plans while n_open still counts the
    // previous round's, so there is nothing to read
    if (a.ctl->err || a.ctl->done) return;
    __shared__ unsigned long long s_m[4];
    const int n_open = a.ctl->n_open;
    unsigned long long m = 0x7FF0000000000000ull;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_open; i += gridDim.x * blockDim.x) {
        unsigned long long b = (unsigned long long)__double_as_longlong(a.p_cost[a.open_out[i]]);
        m = b < m ? b : m;
    }
    for (int o = 32; o > 0; o >>= 1) {
        unsigned long long y = __shfl_down(m, o, 64);
        m = y < m ? y : m;
    }
    // one atomic per workgroup (one per wave on a single word was the
    // kernel's cost: 0.23 ms a round on the indoor query)
    if ((threadIdx.x & 63) == 0) s_m[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w) m = s_m[w] < m ? s_m[w] : m;
        if (m != 0x7FF0000000000000ull) atomicMin(&a.ctl->min_cost_bits, m);
    }
}

__global__ void k_pick_i(RoundArgs a) { pick_next_i(a.ctl, a.h); }

__global__ __launch_bounds__(256) void k_flag_group(RoundArgs a, int32_t* __restrict__ deg) {
    const int n_open = a.ctl->n_open;
    if (a.ctl->done) return;
    const double thr = (double)a.ctl->i * a.h;
    int stop = 0;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_open; i += gridDim.x * blockDim.x) {
        stop |= flag_group_one(a, i, thr) ? 1 : 0;
        int d = 0;
        if (a.o_inB[i]) {
            const int h = a.p_head[a.open_out[i]];
            d = a.row_ptr[h + 1] - a.row_ptr[h];
        }
        deg[i] = d;
    }
    if (__any(stop) && (threadIdx.x & 63) == 0) atomicOr(&a.ctl->goal_stop, 1);
}

// The group in open-list order and its pair offsets (o_keep and deg scanned).
__global__ __launch_bounds__(256) void k_scatter_group(RoundArgs a, const int32_t* deg) {
    const int n_open = a.ctl->n_open;
    if (a.ctl->done) return;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_open; i += gridDim.x * blockDim.x) {
        if (!a.o_inB[i]) continue;
        const int pos = a.o_keep[i];
        a.b_ids[pos] = a.open_out[i];
        a.b_off[pos] = deg[i];
    }
}

__global__ void k_group_finalize(RoundArgs a) {
    Ctl* c = a.ctl;
    c->last_wide = c->wide;
    c->wide = 0;
    if (c->done) {
        c->n_B = 0;
        c->n_pairs = 0;
        return;
    }
    c->n_B = c->scan_total[2];
    c->n_pairs = c->scan_total[3];
    c->n_tasks = 0;
    a.b_off[c->n_B] = c->n_pairs;
    c->done = c->goal_stop ? 1 : 0;
}

void launch_next_group(hipStream_t s, const RoundArgs& a, int32_t n_open_upper, int32_t* deg,
                       int32_t* blk) {
    int b = (n_open_upper + 255) / 256;
    if (b < 1) b = 1;
    if (b > 16384) b = 16384;
    // (the bound counts this round's pairs too; the open list is much
    // shorter, so the minimum strides over it with at most 512 workgroups)
    k_open_min<<<b < 512 ? b : 512, 256, 0, s>>>(a);
    k_pick_i<<<1, 1, 0, s>>>(a);
    k_flag_group<<<b, 256, 0, s>>>(a, deg);
    // (places in the group and pair offsets, both over the open list)
    const ScanJob off{deg, deg, &a.ctl->n_open, &a.ctl->scan_total[3], nullptr, blk + 65536};
    scan_exclusive2(s, ScanJob{a.o_keep, a.o_keep, &a.ctl->n_open, &a.ctl->scan_total[2], nullptr, blk}, &off,
                    n_open_upper);
    k_scatter_group<<<b, 256, 0, s>>>(a, deg);
    k_group_finalize<<<1, 1, 0, s>>>(a);
}

}  // namespace pump
