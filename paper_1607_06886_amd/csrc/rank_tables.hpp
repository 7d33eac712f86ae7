// Rank tables of the particle deviations, and the box test of a pair's
// particles by rank (A4-A6 for the box model).
//
// At plan step s a particle j sits at nom + D[s][.][j]; whether it lies
// between a box's faces on an axis depends on D[s][a][j] alone, and
// fl(nom + v) never decreases with v.  So with the particles of a (step,
// axis) column in ascending order, those at or past the lower face are a tail
// and those not past the upper face a head of the order, and each face takes
// one search for its rank instead of a test per particle.  The tables hold,
// per (step, axis) column,
//   rank row    the N deviations in ascending order (NaN as +inf, last), then
//               a table over N equal cells of the column's span: the rank at
//               which each cell starts.  A search is one load of that rank
//               and one window of eight values from there (about one particle
//               falls in a cell, two and a half in the densest);
//   prefix row  for each rank r the N-bit set of the r first particles.
// A box's hits at a waypoint are the AND over its faces of a prefix set or
// its complement.  A rank is settled by the FP64 comparison of a per-particle
// test (fl(fl(nom + v) - face) against 0), so the hits are the same bits.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "pump_internal.hpp"

namespace pump {

// Floats of one rank row: the values, then N 16-bit ranks.
__host__ __device__ constexpr int rank_row(int N) { return N + N / 2; }
__host__ __device__ constexpr size_t rank_floats(int S1, int N) { return (size_t)S1 * 3 * rank_row(N); }
__host__ __device__ constexpr size_t prefix_words(int S1, int N) {
    return (size_t)S1 * 3 * (N + 1) * (N / 32);
}

// Cell of value x in a column whose values span [mn, mx]: non-decreasing in x,
// so a value of a lower cell is less and one of a higher cell greater.  (A span
// that is empty or not finite has every value in cell 0.)
struct RankCells {
    float mn, scale;
    int top;
    __device__ __forceinline__ RankCells(int N, float lo, float hi)
        : mn(lo), scale(hi > lo && hi - lo < 1e30f ? (float)N / (hi - lo) : 0.0f), top(N - 1) {}
    __device__ __forceinline__ int of(float x) const {
        return (int)fminf(fmaxf((x - mn) * scale, 0.0f), (float)top);
    }
};

// LDS of rank_tables_dev (keys and ranks are read 16 bytes at a time).
struct alignas(16) RankLds {
    uint32_t key[256];
    float sorted[256];
    int rank[256];
};
static_assert(offsetof(RankLds, rank) % 16 == 0, "16-byte reads of the ranks");

// The tables of 256 / N columns by one workgroup of 256 threads, thread c * N
// + j on particle j of the workgroup's column c.  cloud: the columns' spans.
// *has_nan gets 1 when a deviation is NaN (such a particle is in no prefix set;
// zeroed before).
__device__ __forceinline__ void rank_tables_dev(const float* __restrict__ D,
                                                const float* __restrict__ cloud, float* __restrict__ rank,
                                                uint32_t* __restrict__ prefix,
                                                int32_t* __restrict__ has_nan, int N, int S1,
                                                int block, RankLds& s) {
    const int t = threadIdx.x, c = t / N, j = t - c * N, W = N / 32;
    const int col = block * (256 / N) + c;
    const bool on = col < S1 * 3;
    const float v = on ? D[(size_t)col * N + j] : 0.0f;
    // order-preserving integer keys, -0 as +0 and NaN past +inf: a particle's
    // rank is the number of smaller keys, and of equal ones before it
    const bool nan = v != v;
    const uint32_t u = __float_as_uint(v + 0.0f);
    const uint32_t key = nan ? 0xFFFFFFFFu : (u & 0x80000000u ? ~u : u | 0x80000000u);
    if (nan) atomicOr(has_nan, 1);
    s.key[t] = key;
    __syncthreads();
    const uint4* ck = reinterpret_cast<const uint4*>(s.key + c * N);
    int r = 0;
    for (int i = 0; i < N / 4; ++i) {
        const uint4 w = ck[i];
        r += (w.x < key ? 1 : 0) + (w.y < key ? 1 : 0) + (w.z < key ? 1 : 0) + (w.w < key ? 1 : 0);
        if (w.x == key || w.y == key || w.z == key || w.w == key)
            r += (w.x == key && 4 * i < j ? 1 : 0) + (w.y == key && 4 * i + 1 < j ? 1 : 0) +
                 (w.z == key && 4 * i + 2 < j ? 1 : 0) + (w.w == key && 4 * i + 3 < j ? 1 : 0);
    }
    s.sorted[c * N + r] = nan ? INFINITY : v;
    s.rank[t] = nan ? N : r;   // (prefix sets take the particles below their rank)
    __syncthreads();
    if (!on) return;
    float* row = rank + (size_t)col * rank_row(N);
    row[j] = s.sorted[t];
    // cells after the one of the particle of rank j - 1, up to its own, start
    // at rank j
    {
        const float* cl = cloud + (size_t)(col / 3) * 6 + col % 3;
        const RankCells cells(N, cl[0], cl[3]);
        uint16_t* start = reinterpret_cast<uint16_t*>(row + N);
        const int mine = cells.of(s.sorted[t]);
        const int prev = j > 0 ? cells.of(s.sorted[t - 1]) : -1;
        for (int k = prev + 1; k <= mine; ++k) start[k] = (uint16_t)j;
        if (j == N - 1)
            for (int k = mine + 1; k < N; ++k) start[k] = (uint16_t)N;
    }
    // prefix set of rank j, and (threads 0 .. W-1 of the column) of rank N
    const int4* cr = reinterpret_cast<const int4*>(s.rank + c * N);
    uint32_t* m = prefix + (size_t)col * (N + 1) * W;
    auto word = [&](int w, int rk) {
        uint32_t b = 0u;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int4 q = cr[8 * w + i];
            // (q < rk as the sign bit of q - rk)
            b |= ((uint32_t)(q.x - rk) >> 31) << (4 * i) | ((uint32_t)(q.y - rk) >> 31) << (4 * i + 1) |
                 ((uint32_t)(q.z - rk) >> 31) << (4 * i + 2) | ((uint32_t)(q.w - rk) >> 31) << (4 * i + 3);
        }
        return b;
    };
    for (int w = 0; w < W; ++w) m[(size_t)j * W + w] = word(w, j);
    if (j < W) m[(size_t)N * W + j] = word(j, N);
}

// Number of a column's particles with fl(nom + v) < face (upper false) or
// <= face (true); sets `close` when one of them lies within kFlagEps of the
// face.  The search compares in FP32 against face - nom; then the values on
// either side of the rank are taken in FP64 and the rank moves until those
// before the face are before it and the others are not (a step in FP32 can
// only be off among values within rounding of the face).
template <int N>
__device__ __forceinline__ int face_rank(const float* __restrict__ row, const RankCells& cells,
                                         double nom, double face, bool upper, bool& close) {
    typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
    const float t = (float)(face - nom);
    const int start = reinterpret_cast<const uint16_t*>(row + N)[cells.of(t)];
    int base = min(max(start - 1, 0), N - 8), cnt;
    float v[8];
    for (;;) {   // (a second window only where a cell holds more than seven)
        const float4u a = *reinterpret_cast<const float4u*>(row + base);
        const float4u b = *reinterpret_cast<const float4u*>(row + base + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
        cnt = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) cnt += v[i] < t ? 1 : 0;
        if (cnt < 8 || base == N - 8) break;
        base = min(base + 7, N - 8);
    }
    float vl = 0.0f, vh = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        vl = i == cnt - 1 ? v[i] : vl;
        vh = i == cnt ? v[i] : vh;
    }
    int r = base + cnt;
    auto off = [&](float x) { return (nom + (double)x) - face; };
    auto before = [&](double d) { return upper ? d <= 0.0 : d < 0.0; };
    double lo = r > 0 ? off(vl) : -INFINITY, hi = r < N ? off(vh) : INFINITY;
    while (!before(lo)) {
        hi = lo;
        --r;
        lo = r > 0 ? off(row[r - 1]) : -INFINITY;
    }
    while (before(hi)) {
        lo = hi;
        ++r;
        hi = r < N ? off(row[r]) : INFINITY;
    }
    close |= -lo < kFlagEps || hi < kFlagEps;
    return r;
}

}  // namespace pump
