// FP64 device math of the double-integrator connection (Sec. II cost c,
// Sec. IV Cost / Collision primitives).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

namespace pump {

constexpr int kMaxObsWords = 4;   // 64-bit words of a box bit set (256 boxes)

// A value all lanes hold, in scalar registers (loads through a query's record
// are not known to be uniform).
template <typename T>
__device__ __forceinline__ T uniform(T v) {
    static_assert(sizeof(T) % 4 == 0, "whole words");
    uint32_t w[sizeof(T) / 4];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 4; ++i) w[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)w[i]);
    __builtin_memcpy(&v, w, sizeof(T));
    return v;
}

// Boundary sums of a connection x0 -> x1:
//   S_PP = sum P_a^2, S_Pv = sum P_a (v0_a + v1_a), S_vv = sum v0^2 + v0 v1 + v1^2
// with P = p1 - p0.  The minimum-effort cost of duration tau is
//   c(tau) = tau + r (12 S_PP / tau^3 - 12 S_Pv / tau^2 + 4 S_vv / tau).
struct BSums {
    double pp, pv, vv;
};

// boundary_sums and cost_of round every operation on its own (no fused
// multiply-adds), so that each kernel that inlines them -- the near stage's
// steering, the edge costs of pass 2, the batched engine's -- gets the same
// bits from the same inputs.
__device__ __forceinline__ BSums boundary_sums(const float* x0, const float* x1) {
#pragma clang fp contract(off)
    BSums s{0.0, 0.0, 0.0};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double P = (double)x1[a] - (double)x0[a];
        double v0 = (double)x0[3 + a];
        double v1 = (double)x1[3 + a];
        s.pp += P * P;
        s.pv += P * (v0 + v1);
        s.vv += v0 * v0 + v0 * v1 + v1 * v1;
    }
    return s;
}

__device__ __forceinline__ double cost_of(double t, const BSums& s, double r) {
#pragma clang fp contract(off)
    const double it = 1.0 / t;
    return t + r * (it * (it * (12.0 * s.pp * it - 12.0 * s.pv) + 4.0 * s.vv));
}

// a / b for a Newton or Halley step: the hardware reciprocal refined by one
// Newton step (relative error far below what the step needs; the iteration's
// fixed point, where the numerator vanishes, does not depend on it).
__device__ __forceinline__ double step_div(double a, double b) {
    double r = __builtin_amdgcn_rcp(b);
    r = fma(fma(-b, r, 1.0), r, r);
    return a * r;
}

// An upper bound of the cube root of x >= 0 (for root bounds, where any
// larger value also bounds): an FP32 estimate raised by 0.1 %, far above its
// error; below 1e-30 the bound 1e-10, above 1e30 the FP64 cube root.
__device__ __forceinline__ double cbrt_upper(double x) {
    if (!(x >= 1e-30)) return 1e-10;
    if (x > 1e30) return cbrt(x);
    return (double)exp2f(log2f((float)x) * (1.0f / 3.0f)) * 1.001;
}

// Stationarity of c: f(t) = t^4 + a2 t^2 + a1 t + a0 with a2 = -4 r S_vv <= 0,
// a1 = 24 r S_Pv, a0 = -36 r S_PP <= 0; f' = 4 t^3 + 2 a2 t + a1, f'' = 12 t^2 + 2 a2.
struct Quartic {
    double a2, a1, a0;
    __device__ double f(double t) const { return ((t * t + a2) * t + a1) * t + a0; }
    __device__ double g(double t) const { return (4.0 * t * t + 2.0 * a2) * t + a1; }
    __device__ double gp(double t) const { return 12.0 * t * t + 2.0 * a2; }
};

// Root of a function monotone on [lo, hi] whose values at the ends have
// opposite signs: Halley steps (cubic convergence) from the end where
// h * h'' > 0, kept inside the shrinking bracket (bisection when a step
// leaves it); stops once a step moves t by at most 4 ulp.  `which` selects f
// (0) or f' (1) of the quartic.
__device__ __forceinline__ double bracket_root(const Quartic& q, int which, double lo, double hi) {
    auto h0 = [&](double t) { return which ? q.g(t) : q.f(t); };
    auto h1 = [&](double t) { return which ? q.gp(t) : q.g(t); };
    auto h2 = [&](double t) { return which ? 24.0 * t : q.gp(t); };
    double flo = h0(lo);
    double fhi = h0(hi);
    if (flo == 0.0) return lo;
    if (fhi == 0.0) return hi;
    if ((flo < 0.0) == (fhi < 0.0)) return fabs(flo) < fabs(fhi) ? lo : hi;
    const bool rising = flo < 0.0;
    double t = flo * h2(lo) > 0.0 ? lo : (fhi * h2(hi) > 0.0 ? hi : 0.5 * (lo + hi));
    for (int it = 0; it < 200; ++it) {
        const double v = h0(t);
        if (v == 0.0) return t;
        if ((v < 0.0) == rising) lo = t; else hi = t;
        const double d = h1(t);
        const double tn = t - step_div(2.0 * v * d, 2.0 * d * d - v * h2(t));
        if (fabs(tn - t) <= 4.0 * 2.220446049250313e-16 * fabs(t)) return tn;
        const double tb = (tn > lo && tn < hi) ? tn : 0.5 * (lo + hi);
        if (tb == t || !(hi > lo)) break;
        // stop once the bracket is down to a few ulps
        if (hi - lo <= 4.0 * 2.220446049250313e-16 * hi) { t = tb; break; }
        t = tb;
    }
    return t;
}

// Optimal duration and cost of the connection x0 -> x1 (FP64).  The global
// minimiser of c over tau > 0 is one of the upward zero crossings of f
// (local minima of c).  f is concave on (0, ti) and convex on (ti, inf) with
// ti = sqrt(-a2/6), so f' has at most one zero t1 on (0, ti) (only when
// f'(0) = a1 > 0) and one zero t2 on (ti, inf); the upward crossings lie in
// (0, t1) and (t2, inf).  Identical states give tau = cost = 0.
__device__ __forceinline__ void steer64(const float* x0, const float* x1, double r,
                                        double& tau, double& cost) {
    BSums s = boundary_sums(x0, x1);
    if (s.pp == 0.0 && s.vv == 0.0) { tau = 0.0; cost = 0.0; return; }
    Quartic q{-4.0 * r * s.vv, 24.0 * r * s.pv, -36.0 * r * s.pp};
    // Fujiwara bound on the roots of f and of f'/4
    // (cube roots raised to an upper bound: the bounds only need to bound)
    double Bf = 2.0 * fmax(fmax(sqrt(fabs(q.a2)), cbrt_upper(fabs(q.a1))), sqrt(sqrt(0.5 * fabs(q.a0))));
    double Bg = 2.0 * fmax(sqrt(0.5 * fabs(q.a2)), cbrt_upper(0.25 * fabs(q.a1)));
    double ti = sqrt(-q.a2 * (1.0 / 6.0));
    double cand[2];
    int nc = 0;
    if (q.g(ti) >= 0.0) {
        cand[nc++] = bracket_root(q, 0, 0.0, Bf);
    } else {
        double t2 = bracket_root(q, 1, ti, fmax(Bg, ti));
        if (q.f(t2) < 0.0) cand[nc++] = bracket_root(q, 0, t2, fmax(Bf, t2));
        if (q.a1 > 0.0) {
            double t1 = bracket_root(q, 1, 0.0, ti);
            if (q.f(t1) > 0.0) cand[nc++] = bracket_root(q, 0, 0.0, t1);
        }
    }
    double bt = 0.0, bc = INFINITY;
    for (int k = 0; k < nc; ++k) {
        double t = cand[k];
        if (!(t > 0.0)) continue;
        double c = cost_of(t, s, r);
        if (c < bc || (c == bc && t < bt)) { bc = c; bt = t; }
    }
    tau = bt;
    cost = bc;
}

// Rejection test for Near: true only if c(tau) > R for every tau > 0, so the
// pair cannot be an edge with c* < R.  For tau >= R, c(tau) >= tau >= R.  On
// (0, R), c(tau) < R iff g(tau) = tau^3 (c(tau) - R) < 0 with
//   g(tau) = tau^4 - R tau^3 + 4 r S_vv tau^2 - 12 r S_Pv tau + 12 r S_PP.
// A polynomial whose Bernstein coefficients on an interval are all positive is
// positive there.  The coefficients of g / (12 r) on [0, R] come from three
// sums (near_bern32: the first look, 28 operations), and those the bound does
// not settle are split into halves and quarters (de Casteljau, near_split32).
//
// In FP32: every coefficient, also of the parts, is within some 20 units of
// 2^-24 of the magnitudes that enter it, far below the margin of 1e-4 times
// their sum (for those of S_Pv, whose terms can cancel,
// sum |P sv| <= (S_PP + sum sv^2) / 2 and sum sv^2 <= 4/3 S_vv).  What it
// keeps, the steering decides.
struct Near32 {
    float p1, p2, p3, p4;      // R / 4, R / 2, 3 R / 4, R: weights of S_Pv
    float w2, w3, w4, c3;      // weights of S_vv and the constant of b3
    float mp, mv, mc;          // the margin's
};

__device__ __forceinline__ Near32 near32(float r, float R) {
    const float R2 = R * R, q = R2 * R2 / (12.0f * r);
    Near32 k;
    k.p1 = 0.25f * R;
    k.p2 = 0.5f * R;
    k.p3 = 0.75f * R;
    k.p4 = R;
    k.w2 = R2 * (1.0f / 18.0f);
    k.w3 = R2 * (1.0f / 6.0f);
    k.w4 = R2 * (1.0f / 3.0f);
    k.c3 = -0.25f * q;
    k.mp = 1e-4f * (1.0f + 0.5f * R);
    k.mv = 1e-4f * (k.w4 + (2.0f / 3.0f) * R);
    k.mc = 2e-4f * q;
    return k;
}

struct Sums32 {
    float pp, pv, vv;
};

__device__ __forceinline__ Sums32 near_sums32(const float* x0, const float* x1) {
    Sums32 s{0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float P = x1[a] - x0[a], v0 = x0[3 + a], v1 = x1[3 + a], sv = v0 + v1;
        s.pp = fmaf(P, P, s.pp);
        s.pv = fmaf(P, sv, s.pv);
        s.vv = fmaf(v1, sv, fmaf(v0, v0, s.vv));
    }
    return s;
}

__device__ __forceinline__ float min5(const float* b) {
    return fminf(fminf(fminf(b[0], b[1]), fminf(b[2], b[3])), b[4]);
}

// Coefficients on [0, R] and the margin; true: all above it.
__device__ __forceinline__ bool near_bern32(const Near32& k, const Sums32& s, float* b, float& m) {
    b[0] = s.pp;
    b[1] = fmaf(-k.p1, s.pv, s.pp);
    b[2] = fmaf(k.w2, s.vv, fmaf(-k.p2, s.pv, s.pp));
    b[3] = fmaf(k.w3, s.vv, fmaf(-k.p3, s.pv, s.pp)) + k.c3;
    b[4] = fmaf(k.w4, s.vv, fmaf(-k.p4, s.pv, s.pp));
    m = fmaf(k.mp, s.pp, fmaf(k.mv, s.vv, k.mc));
    return min5(b) > m;
}

__device__ __forceinline__ void bern_split(const float* b, float* L, float* Rr) {
    float c[5] = {b[0], b[1], b[2], b[3], b[4]};
    L[0] = c[0];
    Rr[4] = c[4];
#pragma unroll
    for (int lvl = 1; lvl <= 4; ++lvl) {
#pragma unroll
        for (int i = 0; i <= 4 - lvl; ++i) c[i] = 0.5f * (c[i] + c[i + 1]);
        L[lvl] = c[0];
        Rr[4 - lvl] = c[4 - lvl];
    }
}

__device__ __forceinline__ bool near_split32(const float* b, float m) {
    float h[2][5];
    bern_split(b, h[0], h[1]);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (min5(h[k]) > m) continue;
        float q0[5], q1[5];
        bern_split(h[k], q0, q1);
        if (!(fminf(min5(q0), min5(q1)) > m)) return false;
    }
    return true;
}

__device__ __forceinline__ bool surely_not_near(const float* x0, const float* x1, float r, float R) {
    float b[5], m;
    return near_bern32(near32(r, R), near_sums32(x0, x1), b, m) || near_split32(b, m);
}

// Whether steer64 likely takes its one-root branch (f' >= 0 at the inflection
// point): only sorts the work, either branch is there for every pair.
__device__ __forceinline__ bool likely_one_root(const Sums32& s, float r) {
    const float ti = sqrtf(4.0f * r * s.vv * (1.0f / 6.0f));
    return 24.0f * r * s.pv >= (16.0f / 3.0f) * r * s.vv * ti;
}

// Minimum-effort nominal trajectory per axis (cubic Hermite):
//   p(t) = p0 + v0 t + c2 t^2 + c3 t^3,
//   c2 = (3P - (2 v0 + v1) tau) / tau^2,  c3 = (-2P + (v0 + v1) tau) / tau^3.
struct Cubic {
    double c0, c1, c2, c3;
    __device__ double at(double t) const { return c0 + t * (c1 + t * (c2 + t * c3)); }
    __device__ double slope(double t) const { return c1 + t * (2.0 * c2 + t * 3.0 * c3); }
};

// 1 / b from the hardware reciprocal and two Newton steps: within an ulp or
// two of the rounded quotient, for values that need no exact rounding.
__device__ __forceinline__ double recip_fast(double b) {
    double r = __builtin_amdgcn_rcp(b);
    r = fma(fma(-b, r, 1.0), r, r);
    return fma(fma(-b, r, 1.0), r, r);
}

// One axis's coefficients from its (p, v) at the ends, with it = 1 / tau given.
__device__ __forceinline__ Cubic hermite_axis(float p0f, float v0f, float p1f, float v1f, double tau, double it) {
    const double it2 = it * it, it3 = it2 * it;
    const double p0 = (double)p0f, v0 = (double)v0f, v1 = (double)v1f;
    const double P = (double)p1f - p0;
    return Cubic{p0, v0, (3.0 * P - (2.0 * v0 + v1) * tau) * it2, (-2.0 * P + (v0 + v1) * tau) * it3};
}

__device__ __forceinline__ void hermite_r(const float* x0, const float* x1, double tau, double it,
                                          Cubic* out) {
#pragma unroll
    for (int a = 0; a < 3; ++a) out[a] = hermite_axis(x0[a], x0[3 + a], x1[a], x1[3 + a], tau, it);
}

__device__ __forceinline__ void hermite(const float* x0, const float* x1, double tau, Cubic* out) {
    hermite_r(x0, x1, tau, 1.0 / tau, out);   // one division for all six coefficients
}

// Interior stationary points of a cubic on (0, tau), ascending; returns count.
__device__ __forceinline__ int stationary_points(const Cubic& c, double tau, double* br) {
    double A = 3.0 * c.c3, B = 2.0 * c.c2, C = c.c1;
    double r0 = NAN, r1 = NAN;
    if (A == 0.0) {
        if (B != 0.0) r0 = -C / B;
    } else {
        double disc = B * B - 4.0 * A * C;
        if (disc >= 0.0) {
            double sq = sqrt(disc);
            double qv = -0.5 * (B + (B >= 0.0 ? sq : -sq));
            if (qv != 0.0) { r0 = qv / A; r1 = C / qv; }
            else { r0 = 0.0; }
        }
    }
    const bool in0 = r0 > 0.0 && r0 < tau, in1 = r1 > 0.0 && r1 < tau;
    const bool swap = in0 && in1 && r1 < r0;
    br[0] = in0 && !swap ? r0 : r1;
    br[1] = swap ? r0 : r1;
    return (int)in0 + (int)in1;
}

// On a monotone piece [ta, tb] bracketing `level`: the crossing as a bracket
// (lo, hi) with p(lo) on the start side of the level and p(hi) past it.
// Up to 8 Newton steps kept inside the shrinking bracket (bisection when a
// step leaves it); once a step moves t by at most 4 ulp the bracket is
// closed by testing t -/+ 8 ulp.  Otherwise (slow convergence, e.g. a level
// grazing a stationary point) the bracket is bisected until it is a few ulp
// wide (at most 64 halvings).
__device__ __forceinline__ void crossing(const Cubic& c, double ta, double tb, double level,
                                         bool rising, double& lo, double& hi) {
    constexpr double kEps = 2.220446049250313e-16;
    lo = ta; hi = tb;
    auto on_start = [&](double t) {
        const bool below = c.at(t) < level;
        return rising ? below : !below;
    };
    double t = 0.5 * (lo + hi);
    bool conv = false;
    for (int it = 0; it < 8; ++it) {
        const double p = c.at(t);
        const bool below = p < level;
        if (rising ? below : !below) lo = t; else hi = t;
        const double d = c.c1 + t * (2.0 * c.c2 + 3.0 * c.c3 * t);
        double tn = t - (p - level) / d;
        if (!(tn >= lo && tn <= hi)) tn = 0.5 * (lo + hi);
        if (fabs(tn - t) <= 4.0 * kEps * fabs(t)) {
            t = tn;
            conv = true;
            break;
        }
        t = tn;
    }
    if (conv) {
        const double dl = 8.0 * kEps * fmax(fabs(t), 1e-300);
        const double a = fmax(t - dl, ta), b = fmin(t + dl, tb);
        if (on_start(a) && !on_start(b)) {
            lo = fmax(lo, a);
            hi = fmin(hi, b);
            return;
        }
    }
    for (int it = 0; it < 64 && hi - lo > 2.0 * kEps * fabs(hi); ++it) {
        const double mid = 0.5 * (lo + hi);
        if (on_start(mid)) lo = mid; else hi = mid;
    }
}

// The set {t in [0, tau] : lo <= p(t) <= hi} is up to 3 closed intervals, one
// per monotone piece between the stationary points: that of piece k = 0 .. 2 as
// [s, e], or [inf, -inf] where there is none.
__device__ __forceinline__ void slab_piece(const Cubic& c, double tau, double lo, double hi, int k,
                                           double& s, double& e) {
    double br[2];
    const int nb = stationary_points(c, tau, br);
    const double e1 = nb > 0 ? br[0] : tau, e2 = nb > 1 ? br[1] : tau;
    s = INFINITY;
    e = -INFINITY;
    if (k > nb) return;
    const double ta = k == 0 ? 0.0 : (k == 1 ? e1 : e2);
    const double tb = k == nb ? tau : (k == 0 ? e1 : e2);
    const double pa = c.at(ta), pb = c.at(tb);
    const bool rising = pb >= pa;
    const double pmin = fmin(pa, pb), pmax = fmax(pa, pb);
    if (!(pmax >= lo && pmin <= hi)) return;
    double l0, l1, h0, h1;
    if (rising) {
        if (pmin >= lo) s = ta; else { crossing(c, ta, tb, lo, true, l0, l1); s = l1; }
        if (pmax <= hi) e = tb; else { crossing(c, ta, tb, hi, true, h0, h1); e = h0; }
    } else {
        if (pmax <= hi) s = ta; else { crossing(c, ta, tb, hi, false, h0, h1); s = h1; }
        if (pmin >= lo) e = tb; else { crossing(c, ta, tb, lo, false, l0, l1); e = l0; }
    }
}

// Range of a cubic over [0, tau] (endpoints and stationary points).
__device__ __forceinline__ void cubic_range(const Cubic& c, double tau, double& mn, double& mx) {
    double br[2];
    int nb = stationary_points(c, tau, br);
    double p0 = c.at(0.0), p1 = c.at(tau);
    mn = fmin(p0, p1); mx = fmax(p0, p1);
    for (int k = 0; k < nb; ++k) { double v = c.at(br[k]); mn = fmin(mn, v); mx = fmax(mx, v); }
}

// Does the nominal trajectory (three axis cubics on [0, tau]) meet the closed
// box? It is inside at time t iff all three coordinates are in their slabs,
// so it meets the box iff the three per-axis in-slab sets (slab_piece)
// intersect: the exact test.
//
// Cheaper tests settle most cases first, over equal pieces of the trajectory
// and their quarters: a sample point (interior piece ends) inside the box
// proves a hit; and on each piece a cubic lies in the hull of its Bernstein
// coefficients p(ta), p(ta) + h p'(ta)/3, p(tb) - h p'(tb)/3, p(tb), so a piece
// whose hull (widened by kHullMargin, far above the rounding of these values)
// misses the box on some axis cannot meet it.  When every piece is cleared the
// trajectory misses the box.  They only settle cases the exact test decides
// the same way.
constexpr double kHullMargin = 1e-9;

// ---------------------------------------------------------------------------
// Half-Space Monte Carlo (Sec. III-B): the local convex region around a
// workspace point y is built one plane at a time.  Each step takes the
// closest point of the remaining boxes (ties: lowest box index), d = that
// point - y, and drops every remaining box that lies in the closed
// half-space d.(z - y) >= d.d (always the box that gave d).  `rem` holds the
// remaining boxes as bits; returns false when none remains.
// ---------------------------------------------------------------------------
// A step for a wave whose lanes hold points of their own (all lanes call it; a
// lane without boxes left only lends its place): boxes that no lane has left are
// passed over, so the others are read once for all lanes.  boxes: FP64 (lo xyz,
// hi xyz).  n_obs at most 64 nw.
__device__ __forceinline__ bool hs_next_lanes(const double* y, const double* boxes, int nw,
                                              unsigned long long* rem, double* d) {
#pragma clang fp contract(off)
    int best = -1;
    double best_d2 = INFINITY;
    double b0 = 0.0, b1 = 0.0, b2 = 0.0;
    unsigned long long any[kMaxObsWords];
#pragma unroll
    for (int w = 0; w < kMaxObsWords; ++w) {
        any[w] = 0ull;
        if (w < nw) {
            unsigned long long u = rem[w];
            for (int o = 32; o > 0; o >>= 1) u |= __shfl_xor(u, o, 64);
            any[w] = u;
        }
    }
#pragma unroll
    for (int w = 0; w < kMaxObsWords; ++w) {
        unsigned long long m = any[w];
        while (m) {
            const int i = __builtin_amdgcn_readfirstlane(__ffsll((long long)m) - 1);
            m &= m - 1ull;
            const double* b = boxes + (w * 64 + i) * 6;
            const double d0 = fmin(fmax(y[0], b[0]), b[3]) - y[0];
            const double d1 = fmin(fmax(y[1], b[1]), b[4]) - y[1];
            const double d2 = fmin(fmax(y[2], b[2]), b[5]) - y[2];
            const double dd = (d0 * d0 + d1 * d1) + d2 * d2;
            if (((rem[w] >> i) & 1ull) && dd < best_d2) {
                best_d2 = dd;
                best = w * 64 + i;
                b0 = d0; b1 = d1; b2 = d2;
            }
        }
    }
    d[0] = b0; d[1] = b1; d[2] = b2;
    const double dd = (b0 * b0 + b1 * b1) + b2 * b2;
    const double dy = (b0 * y[0] + b1 * y[1]) + b2 * y[2];
#pragma unroll
    for (int w = 0; w < kMaxObsWords; ++w) {
        unsigned long long m = any[w];
        while (m) {
            const int i = __builtin_amdgcn_readfirstlane(__ffsll((long long)m) - 1);
            m &= m - 1ull;
            const double* b = boxes + (w * 64 + i) * 6;
            double lo_part = fmin(b0 * b[0], b0 * b[3]);
            lo_part = lo_part + fmin(b1 * b[1], b1 * b[4]);
            lo_part = lo_part + fmin(b2 * b[2], b2 * b[5]);
            if (w * 64 + i == best || lo_part - dy >= dd) rem[w] &= ~(1ull << i);
        }
    }
    if (best < 0)   // (nothing near: a point that is not finite)
        for (int w = 0; w < kMaxObsWords; ++w) rem[w] = 0ull;
    return best >= 0;
}

// The same for a wave whose lanes share y and rem (all 64 lanes call it, in
// uniform control flow): lane l takes box w * 64 + l, the nearest box is the
// wave minimum of the same squared distances, taken at its lowest box index
// (as above, where the first strict minimum in box order is kept), and the
// boxes the new plane removes are one ballot per word.  Every value is the
// same expression as above, so the planes and the boxes left are identical.
__device__ __forceinline__ bool hs_next_wave(const double* y, const double* boxes, int n_obs,
                                             unsigned long long* rem, double* d) {
#pragma clang fp contract(off)
    const int lane = threadIdx.x & 63;
    int best = -1;
    double best_d2 = INFINITY;
    for (int w = 0; w * 64 < n_obs; ++w) {
        double d2 = INFINITY;
        if ((rem[w] >> lane) & 1ull) {
            const double* b = boxes + (w * 64 + lane) * 6;
            double dv[3];
            for (int a = 0; a < 3; ++a)
                dv[a] = fmin(fmax(y[a], b[a]), b[3 + a]) - y[a];
            d2 = (dv[0] * dv[0] + dv[1] * dv[1]) + dv[2] * dv[2];
            if (!(d2 < INFINITY)) d2 = INFINITY;   // never chosen, as in the loop
        }
        double m = d2;
        for (int off = 32; off >= 1; off >>= 1) m = fmin(m, __shfl_xor(m, off, 64));
        if (m < best_d2) {
            best_d2 = m;
            best = w * 64 + __ffsll((long long)__ballot(d2 == m)) - 1;
        }
    }
    if (best < 0) return false;
    double bd[3];
    {
        const double* b = boxes + best * 6;
        for (int a = 0; a < 3; ++a) bd[a] = fmin(fmax(y[a], b[a]), b[3 + a]) - y[a];
    }
    d[0] = bd[0]; d[1] = bd[1]; d[2] = bd[2];
    const double dd = (bd[0] * bd[0] + bd[1] * bd[1]) + bd[2] * bd[2];
    const double dy = (bd[0] * y[0] + bd[1] * y[1]) + bd[2] * y[2];
    for (int w = 0; w * 64 < n_obs; ++w) {
        const int o = w * 64 + lane;
        bool drop = false;
        if ((rem[w] >> lane) & 1ull) {
            const double* b = boxes + o * 6;
            double lo_part = 0.0;
            for (int a = 0; a < 3; ++a)
                lo_part += fmin(bd[a] * b[a], bd[a] * b[3 + a]);
            drop = o == best || lo_part - dy >= dd;
        }
        rem[w] &= ~__ballot(drop);
    }
    return true;
}

// eq. (7): the plane normal made perpendicular to the nominal velocity v
// (unchanged at rest); b = a.a.
__device__ __forceinline__ void hs_project(const double* d, const double* v, double* a, double& b) {
#pragma clang fp contract(off)
    const double vv = (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2];
    if (vv > 0.0) {
        const double f = ((d[0] * v[0] + d[1] * v[1]) + d[2] * v[2]) / vv;
        for (int k = 0; k < 3; ++k) a[k] = d[k] - f * v[k];
    } else {
        for (int k = 0; k < 3; ++k) a[k] = d[k];
    }
    b = (a[0] * a[0] + a[1] * a[1]) + a[2] * a[2];
}

__device__ __forceinline__ void all_boxes(int n_obs, unsigned long long* rem) {
    for (int w = 0; w < kMaxObsWords; ++w) {
        const int lo = w * 64;
        rem[w] = n_obs >= lo + 64 ? ~0ull : (n_obs > lo ? ((1ull << (n_obs - lo)) - 1ull) : 0ull);
    }
}

}  // namespace pump
