// Workspace partition for range queries against the obstacle boxes (the
// broad phase the paper suggests for cluttered maps, Sec. V-C).
//
// Along each axis the span of the boxes is cut into kBins equal bins, with
// bin(x) = clamp(floor((x - org) * scale), 0, kBins - 1), a non-decreasing
// function of x (each floating-point step is monotone).  Per axis and bin b
// two bit sets over the boxes are kept:
//   lo_le[b] = { o : bin(lo_o) <= b },   hi_ge[b] = { o : bin(hi_o) >= b }.
// A box that meets the interval [p, q] on an axis (lo_o <= q, hi_o >= p) has
// bin(lo_o) <= bin(q) and bin(hi_o) >= bin(p), so it is in
// lo_le[bin(q)] & hi_ge[bin(p)]; the AND over the three axes is a superset of
// the boxes a 3-D range meets, found with six shared-memory reads per word of
// the bit set.  The exact range test then runs over that superset only, so
// the boxes found are exactly those of a test over every box.
//
// The table is built once per query in device memory, and the kernels that ask
// it copy it to LDS.
#pragma once

#include "device_math.hpp"
#include "pump_internal.hpp"

namespace pump {

constexpr int kBins = 64;

// Layout: 8 header words (org xyz, scale xyz, boxes, words per set), then the
// sets lo_le[3][kBins][nw] and hi_ge[3][kBins][nw].
constexpr int kBinHeader = 8;
__host__ __device__ constexpr int bin_words(int n_obs) {
    return kBinHeader + 2 * 3 * kBins * ((n_obs + 63) / 64) * 2;
}

// One workgroup (n at most kMaxObs); boxes b[o * 6 + (lo xyz, hi xyz)], out: bin_words(n) words.
__device__ __forceinline__ void box_bins_write(const float* __restrict__ b, int n,
                                               uint32_t* __restrict__ out) {
    __shared__ float s_org[3], s_scale[3], s_b[kMaxObs * 6];
    const int nw = (n + 63) / 64;
    for (int t = threadIdx.x; t < n * 6; t += blockDim.x) s_b[t] = b[t];
    __syncthreads();
    if (threadIdx.x < 64) {
        for (int a = 0; a < 3; ++a) {
            float lo = INFINITY, hi = -INFINITY;
            for (int o = threadIdx.x; o < n; o += 64) {
                lo = fminf(lo, s_b[o * 6 + a]);
                hi = fmaxf(hi, s_b[o * 6 + 3 + a]);
            }
            for (int k = 32; k > 0; k >>= 1) {
                lo = fminf(lo, __shfl_xor(lo, k, 64));
                hi = fmaxf(hi, __shfl_xor(hi, k, 64));
            }
            if (threadIdx.x == 0) {
                const bool ok = n > 0 && hi > lo;
                s_org[a] = ok ? lo : 0.0f;   // otherwise every box in bin 0
                s_scale[a] = ok ? (float)kBins / (hi - lo) : 0.0f;
                out[a] = __float_as_uint(s_org[a]);
                out[3 + a] = __float_as_uint(s_scale[a]);
            }
        }
    }
    if (threadIdx.x == 0) {
        out[6] = (uint32_t)n;
        out[7] = (uint32_t)nw;
    }
    __syncthreads();
    const int per = 3 * kBins * nw;
    for (int t = threadIdx.x; t < 2 * per; t += blockDim.x) {
        const bool ge = t >= per;
        const int u = ge ? t - per : t;
        const int w = u % nw, bn = (u / nw) % kBins, a = u / (nw * kBins);
        unsigned long long bits = 0ull;
        for (int k = 0; k < 64 && w * 64 + k < n; ++k) {
            const float x = s_b[(w * 64 + k) * 6 + (ge ? 3 : 0) + a];
            const int bx = (int)fminf(fmaxf((x - s_org[a]) * s_scale[a], 0.0f), (float)(kBins - 1));
            if (ge ? bx >= bn : bx <= bn) bits |= 1ull << k;
        }
        out[kBinHeader + 2 * t] = (uint32_t)bits;
        out[kBinHeader + 2 * t + 1] = (uint32_t)(bits >> 32);
    }
}

// A copy of it in LDS.
struct BinView {
    float org[3], scale[3];
    const unsigned long long* set;   // lo_le, then hi_ge
    int nw;
};

// Candidate boxes (word w) of the bins idx = (bin(hi) on lo_le, bin(lo) on
// hi_ge) per axis.  A range that is not finite needs no case of its own: NaN
// ends fall in bin 0 and meet no box, infinite ones in the end bins.
struct BinRange {
    int le[3], ge[3];
};

__device__ __forceinline__ void bin_range(const BinView& v, const float* lo3, const float* hi3,
                                          BinRange& r) {
    const int per = 3 * kBins * v.nw;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float top = (float)(kBins - 1);
        const int bh = (int)fminf(fmaxf((hi3[a] - v.org[a]) * v.scale[a], 0.0f), top);
        const int bl = (int)fminf(fmaxf((lo3[a] - v.org[a]) * v.scale[a], 0.0f), top);
        r.le[a] = (a * kBins + bh) * v.nw;
        r.ge[a] = per + (a * kBins + bl) * v.nw;
    }
}

__device__ __forceinline__ unsigned long long bin_candidates(const BinView& v, const BinRange& r,
                                                             int w) {
    return v.set[r.le[0] + w] & v.set[r.ge[0] + w] & v.set[r.le[1] + w] & v.set[r.ge[1] + w] &
           v.set[r.le[2] + w] & v.set[r.ge[2] + w];
}

}  // namespace pump
