// ara_math.h -- device arithmetic of secondary uncertainty (section 3 of the
// paper): Philox4x32-10 draws, the normal mix of section 3.2 and the inverse
// regularized incomplete beta of section 3.3, in an FP32 bulk form and an
// FP64 form for the tails and for shapes the FP32 form does not cover.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ara_internal.h"

namespace ara {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).  The ten round keys are
// the same for every draw of a run, so the host expands them once
// (PhiloxKeys) and the device only runs the rounds.
// ---------------------------------------------------------------------------
struct PhiloxKeys {
    uint32_t k0, k1;           // the key; round r uses (k0 + r W0, k1 + r W1)
};

constexpr uint32_t kPhiloxM0 = 0xD2511F53u;
constexpr uint32_t kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u;
constexpr uint32_t kPhiloxW1 = 0xBB67AE85u;

inline PhiloxKeys philox_keys(uint64_t seed) {
    PhiloxKeys k;
    k.k0 = (uint32_t)seed;
    k.k1 = (uint32_t)(seed >> 32);
    return k;
}

// a ^ b ^ c in one instruction; the compiler makes two of it, 20 more for a draw (1M trials
// x 16 ELTs, the lean pass: 8.49 -> 8.28 ms).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// The key is wave-uniform, so its schedule runs on the scalar unit.
__device__ __forceinline__ uint4 philox10(uint4 c, const PhiloxKeys &k) {
    uint32_t k0 = k.k0, k1 = k.k1;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        uint64_t p0 = (uint64_t)kPhiloxM0 * (uint64_t)c.x;
        uint64_t p1 = (uint64_t)kPhiloxM1 * (uint64_t)c.z;
        uint4 n;
        n.x = xor3((uint32_t)(p1 >> 32), c.y, k0);
        n.y = (uint32_t)p1;
        n.z = xor3((uint32_t)(p0 >> 32), c.w, k1);
        n.w = (uint32_t)p0;
        c = n;
        k0 += kPhiloxW0;
        k1 += kPhiloxW1;
    }
    return c;
}

// Word 0 only: the last round's x output needs only the product M1 * c.z.
__device__ __forceinline__ uint32_t philox10_x0(uint4 c, const PhiloxKeys &k) {
    uint32_t k0 = k.k0, k1 = k.k1;
#pragma unroll
    for (int r = 0; r < 9; ++r) {
        uint64_t p0 = (uint64_t)kPhiloxM0 * (uint64_t)c.x;
        uint64_t p1 = (uint64_t)kPhiloxM1 * (uint64_t)c.z;
        uint4 n;
        n.x = xor3((uint32_t)(p1 >> 32), c.y, k0);
        n.y = (uint32_t)p1;
        n.z = xor3((uint32_t)(p0 >> 32), c.w, k1);
        n.w = (uint32_t)p0;
        c = n;
        k0 += kPhiloxW0;
        k1 += kPhiloxW1;
    }
    return xor3(__umulhi(kPhiloxM1, c.z), c.y, k0);
}

// Odd multiple of 2^-24: u = ((w >> 8) | 1) * 2^-24, so 1 - u is exact too.
// Returns the 24-bit odd integer j; u = j * 2^-24.
__device__ __forceinline__ uint32_t u24(uint32_t w) { return (w >> 8) | 1u; }

// ---------------------------------------------------------------------------
// FP32 building blocks
// ---------------------------------------------------------------------------
__device__ __forceinline__ float rcp_f(float x) { return __builtin_amdgcn_rcpf(x); }

// Reciprocal with one Newton step (about 0.5 ulp): cheaper than an IEEE
// division where the last half ulp does not matter.
__device__ __forceinline__ float rcp_nr(float y) {
    const float r = rcp_f(y);
    return r * fmaf(-y, r, 2.0f);
}

// log2(1 - x) for 0 <= x < 1: w = 1 - x rounds, but its rounding error
// e = (1 - w) - x is exact (Fast2Sum, |1| >= |x|), and
// log2(1 - x) = log2(w) + log2(1 + e/w) ~ log2(w) + (e/w) log2(e).
__device__ __forceinline__ float log2_1m(float x, float w) {
    const float e = (1.0f - w) - x;
    return fmaf(e * rcp_f(w), 1.4426950408889634f, __log2f(w));
}

// Continued fraction of DLMF 8.17.22: I_x(a, b) = x^a (1-x)^b / (a B(a,b)) / K
// with K = 1 + d1/(1 + d2/(1 + ...)),
//   d_{2m+1} = -(a+m)(a+b+m) x / ((a+2m)(a+2m+1)),
//   d_{2m}   =  m(b-m) x / ((a+2m-1)(a+2m)).
// Evaluated backward from term n (more accurate in FP32 than the forward
// recurrence) without divisions: with d_j = p_j / q_j and K_j = N_j / D_j,
// N_j = q_j N_{j+1} + p_j D_{j+1}, D_j = q_j N_{j+1}.  Terms go in pairs
// (2m, 2m-1); n (even) comes from the row (enough terms at the slowest
// point of the branch, see cf_terms); lanes with fewer terms than the batch
// maximum nmax (even, wave-uniform) leave their (N, D) at the start value
// until their first term, a select that is skipped when every lane needs
// nmax terms.  Rescaled every pair.  Returns N, D.
__device__ __forceinline__ void beta_cf32(float a, float b, float x, int n, int nmax, float *Nout,
                                          float *Dout) {
    float N = 1.0f, D = 1.0f;
    const float am1 = a - 1.0f, apbm1 = (a + b) - 1.0f;
    // one pair of terms (2m, 2m-1), rescaled to N = 1
    auto pair = [&](float fm, float *Dn) {
        // even term 2m: p = m (b - m) x, q = (a + 2m - 1)(a + 2m) = te (te + 1)
        const float te = fmaf(2.0f, fm, am1);
        const float qe = fmaf(te, te, te);
        const float pe = fm * (b - fm) * x;
        // odd term 2m-1: p = -(a+m-1)(a+b+m-1) x, q = (a+2m-2)(a+2m-1) = (te - 1) te
        const float qo = fmaf(te, te, -te);
        const float po = -(am1 + fm) * (apbm1 + fm) * x;
        const float N1 = fmaf(qe, N, pe * D), D1 = qe * N;
        const float N2 = fmaf(qo, N1, po * D1), D2 = qo * N1;
        *Dn = D2 * rcp_f(N2);
    };
    float fm = (float)(nmax >> 1);           // exact small integer, stepped down exactly
    if (__all(n >= nmax)) {
        // every lane takes every term (the usual case: one shape per batch)
        for (int m = nmax >> 1; m >= 1; --m, fm -= 1.0f) pair(fm, &D);
    } else {
        for (int m = nmax >> 1; m >= 1; --m, fm -= 1.0f) {
            float Dn;
            pair(fm, &Dn);
            const bool on = 2 * m <= n;
            N = on ? 1.0f : N;
            D = on ? Dn : D;
        }
    }
    *Nout = N;
    *Dout = D;
}

// Initial guess: Abramowitz & Stegun 26.2.22 for the upper-tail normal
// deviate y of the smaller tail probability, then A&S 26.5.22 for the Beta
// quantile (valid for a, b > 1/2; used here for a, b >= 1).
__device__ __forceinline__ float beta_guess32(float a, float b, float z, float zc) {
    // only a starting point: approximate reciprocals are enough
    const bool lowz = z < 0.5f;
    const float pp = lowz ? z : zc;
    const float t = sqrtf(-2.0f * __logf(pp));
    float y = t - (2.30753f + 0.27061f * t) * rcp_f(1.0f + t * (0.99229f + 0.04481f * t));
    if (!lowz) y = -y;                       // y = Phi^-1(1 - z)
    const float lam = (y * y - 3.0f) * (1.0f / 6.0f);
    const float ra = rcp_f(2.0f * a - 1.0f), rb = rcp_f(2.0f * b - 1.0f);
    const float rh = 0.5f * (ra + rb);       // 1 / h, h = 2 / (ra + rb)
    const float w = y * sqrtf(rcp_f(rh) + lam) * rh -
                    (rb - ra) * (lam + 5.0f / 6.0f - (2.0f / 3.0f) * rh);
    return a * rcp_f(a + b * __expf(2.0f * w));
}

// One polynomial segment (see kShapeSlots) at its local coordinate.
__device__ __forceinline__ float seg_poly(const float *c, float d) {
    const float4 lo = *reinterpret_cast<const float4 *>(c);
    const float4 hi = *reinterpret_cast<const float4 *>(c + 4);
    float r = fmaf(hi.w, d, hi.z);
    r = fmaf(r, d, hi.y);
    r = fmaf(r, d, hi.x);
    r = fmaf(r, d, lo.w);
    r = fmaf(r, d, lo.z);
    r = fmaf(r, d, lo.y);
    return fmaf(r, d, lo.x);
}

// Octave and mantissa of p = min(j, 2^24 - j) for an odd grid integer j: the
// conversion is exact, so the local coordinate carries no rounding.
__device__ __forceinline__ int grid_octave(uint32_t j, bool *upper, float *d) {
    *upper = j > 8388608u;
    const uint32_t bits = __float_as_uint((float)(*upper ? 16777216u - j : j));
    *d = __uint_as_float((bits & 0x7fffffu) | 0x3f800000u) - 1.5f;
    return (int)(bits >> 23) - 127;
}

// min(z, 1 - z) of the draw z = j 2^-24.
__device__ __forceinline__ float grid_tail(uint32_t j) {
    return (float)min(j, 16777216u - j) * 5.9604644775390625e-08f;
}

// Segment of a slot (offset in floats) and local coordinate of a draw.
__device__ __forceinline__ uint32_t slot_segment(uint32_t j, float *d) {
    bool upper;
    const int e = grid_octave(j, &upper, d);
    return (uint32_t)(kSegCoefs * (e + (upper ? kSegUpper : 0)));
}

// The same of a normal deviate v, |v| <= kDevMax.
__device__ __forceinline__ uint32_t dev_segment(float v, float *d) {
    const float i = rintf(2.0f * v);
    *d = fmaf(2.0f, v, -i);
    return (uint32_t)(kSegCoefs * (kSegDev + min(max((int)i + kDevHalf, 0), kDevSegs - 1)));
}

// The quantile of a slot's shape at the draw z = j 2^-24.
__device__ __forceinline__ float slot_quantile(const float *slot, uint32_t j) {
    float d;
    const uint32_t at = slot_segment(j, &d);
    return seg_poly(slot + at, d);
}

// Phi^-1(j 2^-24) from the normal segments.
__device__ __forceinline__ float norm_dev(const float *norm, uint32_t j) {
    bool upper;
    float d;
    const int e = grid_octave(j, &upper, &d);
    const float v = seg_poly(norm + kSegCoefs * e, d);
    return upper ? -v : v;
}

// The quantile of a slot's shape at z = Phi(v), |v| <= kDevMax.
__device__ __forceinline__ float slot_quantile_dev(const float *slot, float v) {
    float d;
    const uint32_t at = dev_segment(v, &d);
    return seg_poly(slot + at, d);
}

// I_x(a,b) (*I) and 1 - I_x(a,b) (*Ic), each on the side where it is
// accurate, and the prefactor x^a (1-x)^b / B(a,b) (*front; the density is
// front / (x (1-x))); lnb2 = log2 B(a, b); na / nb the continued-fraction
// terms of the (a, b) and (b, a) branches; nmax the wave-uniform bound of both.
__device__ __forceinline__ void beta_inc32(float a, float b, float lnb2, int na, int nb, int nmax,
                                           float x, float *I, float *Ic, float *front_out) {
    const float w = 1.0f - x;
    const float e2 = fmaf(a, __log2f(x), fmaf(b, log2_1m(x, w), -lnb2));
    const float front = exp2f(e2);
    *front_out = front;
    const bool direct = x * (a + b + 2.0f) < a + 1.0f;
    // one loop for both branches: (a, b, x) directly, else (b, a, 1 - x)
    const float A = direct ? a : b, B = direct ? b : a, X = direct ? x : w;
    float N, D;
    beta_cf32(A, B, X, direct ? na : nb, nmax, &N, &D);
    const float v = front * D * rcp_nr(N * A);
    *I = direct ? v : 1.0f - v;
    *Ic = direct ? 1.0f - v : v;
}

// FP32 quantile x = I^-1(z; a, b) given z and zc = 1 - z (both exact), for
// shapes inside the FP32 domain (kF32MinShape <= a, b <= kF32MaxShape).
// Halley iterations on the side where the root is at most ~1/2 (mirroring
// through I_{1-x}(b,a) = 1 - z otherwise), with the residual taken on the
// side of the smaller of z, zc so it never cancels.  The first iteration
// evaluates the continued fraction with about half its terms (the guess is
// only good to ~1e-2, so a residual good to ~1e-4 serves that step); every
// later one uses all of them.  The step sizes use reciprocals (they only set
// the speed, the residual sets the root): with f the density and r the
// residual, u = r / f = r x (1-x) / front and u (log f)' = r ((a-1)(1-x) -
// (b-1) x) / front share one reciprocal.  Stops when every lane's last
// full-accuracy step was below 2^-10 of the root (Halley: the next error ~
// step^3); a lane keeps the iterate of its own first such step, so its
// result does not depend on how many iterations the wavefront runs.  Returns
// false in *ok if it did not converge (the caller then uses the FP64 path).
__device__ __forceinline__ float beta_quantile32(float a, float b, float lnb2, int na, int nb,
                                                 float z, float zc, bool *ok) {
    float x0 = beta_guess32(a, b, z, zc);
    const bool mirror = x0 > 0.5f;
    if (mirror) x0 = 1.0f - x0;
    float A = a, B = b, Z = z, ZC = zc;
    int NA = na, NB = nb;
    if (mirror) {
        A = b; B = a; Z = zc; ZC = z; NA = nb; NB = na;
    }
    // bound of both branches' term counts over the active lanes only (a
    // shuffle would also read the registers of inactive lanes): bitwise
    // maximum by ballots, counts are below 64
    const int nl = max(na, nb);
    int nmax = 0;
#pragma unroll
    for (int bit = 32; bit >= 1; bit >>= 1)
        if (__any(nl >= (nmax | bit))) nmax |= bit;
    const int nhalf = max(2, ((nmax >> 1) + 1) & ~1);
    // this lane's own half count (the wave's bounds only size the loops, so a
    // lane's result does not depend on the lanes beside it)
    const int nh = max(2, ((nl >> 1) + 1) & ~1);
    float x = fminf(fmaxf(x0, 1e-30f), 0.75f);
    const bool lower = Z <= 0.5f;
    const float am1 = A - 1.0f, bm1 = B - 1.0f;
    bool conv = false;
    float xf = x;          // the lane's answer: its iterate at its own first convergence
    for (int it = 0; it < 6; ++it) {
        const int nt = it == 0 ? nhalf : nmax;
        const int nown = it == 0 ? nh : nmax;
        float I, Ic, front;
        beta_inc32(A, B, lnb2, min(NA, nown), min(NB, nown), nt, x, &I, &Ic, &front);
        const float r = lower ? (I - Z) : (ZC - Ic);
        const float w = 1.0f - x;
        const float rf = r * rcp_f(front);
        const float u = rf * (x * w);
        const float uh = rf * fmaf(am1, w, -bm1 * x);
        const float t = u * rcp_f(1.0f - 0.5f * fminf(1.0f, uh));
        float xn = x - t;
        if (!(xn > 0.0f)) xn = 0.5f * x;
        if (!(xn < 1.0f)) xn = 0.5f * (x + 1.0f);
        if (!conv) {
            xf = xn;
            conv = it > 0 && fabsf(xn - x) <= 9.765625e-4f * xn;
        }
        x = xn;
        if (__all(conv)) break;
    }
    *ok = conv && isfinite(xf);
    return mirror ? 1.0f - xf : xf;
}

// ---------------------------------------------------------------------------
// FP64 path (tails, shapes outside the FP32 domain, FP32 non-convergence).
// ---------------------------------------------------------------------------
__device__ inline double beta_cf64(double a, double b, double x) {
    double Am2 = 1.0, Bm2 = 0.0, Am1 = 1.0, Bm1 = 1.0, qprev = 1.0, Kprev = 1.0, K = 1.0;
    const double apb = a + b;
    for (int m = 0; m < 4000; ++m) {
        const double fm = (double)m;
        const double t0 = a + 2.0 * fm;
        const double qo = t0 * (t0 + 1.0);
        const double ao = qprev * (-(a + fm) * (apb + fm) * x);
        const double A1 = qo * Am1 + ao * Am2;
        const double B1 = qo * Bm1 + ao * Bm2;
        const double qe = (t0 + 1.0) * (t0 + 2.0);
        const double ae = qo * ((fm + 1.0) * (b - fm - 1.0) * x);
        const double A2 = qe * A1 + ae * Am1;
        const double B2 = qe * B1 + ae * Bm1;
        qprev = qe;
        const double s = 1.0 / B2;
        Am2 = A1 * s;
        Bm2 = B1 * s;
        Am1 = A2 * s;
        Bm1 = 1.0;
        K = Am1;
        if (fabs(K - Kprev) <= 1e-16 * fabs(K)) break;
        Kprev = K;
    }
    return 1.0 / K;
}

// Pairs of terms (2m - 1, 2m) after which the fraction stays within tol
// (relative) of its limit at the slowest point of its branch,
// x = (a+1)/(a+b+2) (it converges faster for smaller x); 0 when more than
// most are needed.  Evaluated forward in FP64 at load time, once to the limit
// and once to the count: O(n) where evaluating every candidate backward took
// O(n^2) terms (k_fit_rows over 768k rows 0.33 ms before).
__device__ inline int cf_pairs(double a, double b, double tol, int most) {
    const double x = (a + 1.0) / (a + b + 2.0), apb = a + b;
    double ref = 0.0;
    for (int pass = 0; pass < 2; ++pass) {
        double Am2 = 1.0, Bm2 = 0.0, Am1 = 1.0, Bm1 = 1.0, qprev = 1.0, K = 1.0;
        const int last = pass ? most : 2000;
        for (int m = 0; m < last; ++m) {
            const double fm = (double)m, t0 = a + 2.0 * fm;
            const double qo = t0 * (t0 + 1.0), ao = qprev * (-(a + fm) * (apb + fm) * x);
            const double A1 = qo * Am1 + ao * Am2, B1 = qo * Bm1 + ao * Bm2;
            const double qe = (t0 + 1.0) * (t0 + 2.0), ae = qo * ((fm + 1.0) * (b - fm - 1.0) * x);
            const double A2 = qe * A1 + ae * Am1, B2 = qe * B1 + ae * Bm1;
            qprev = qe;
            const double s = 1.0 / B2, Kn = A2 * s;
            Am2 = A1 * s;
            Bm2 = B1 * s;
            Am1 = Kn;
            Bm1 = 1.0;
            if (pass ? fabs(ref / Kn - 1.0) < tol : fabs(Kn - K) <= 1e-15 * fabs(Kn)) {
                if (pass) return m + 1;
                K = Kn;
                break;
            }
            K = Kn;
        }
        ref = K;
    }
    return 0;
}

// Terms the FP32 quantile takes (truncation below 1e-8; even, at most 62).
__device__ inline int cf_terms(double a, double b) { return 2 * cf_pairs(a, b, 1e-8, 31); }

// The fraction backward from a known number of pairs, without divisions (see
// beta_cf32); every pair is scaled by an approximate reciprocal of its N, which
// cancels in the ratio.  About 25 instructions a pair where the forward form
// with its division and its convergence test takes 45.  Returns 1 / K.
__device__ inline double beta_cf64_pairs(double a, double b, double x, int pairs) {
    const double am1 = a - 1.0, apbm1 = (a + b) - 1.0;
    double N = 1.0, D = 1.0, fm = (double)pairs;
    for (int m = pairs; m >= 1; --m, fm -= 1.0) {
        const double te = fma(2.0, fm, am1);
        const double qe = fma(te, te, te), qo = fma(te, te, -te);
        const double mx = fm * x;
        const double pe = (b - fm) * mx;
        const double po = -(am1 + fm) * ((apbm1 + fm) * x);
        const double D1 = qe * N;
        const double N1 = fma(pe, D, D1);
        const double D2 = qo * N1;
        const double N2 = fma(po, D1, D2);
        const double s = __builtin_amdgcn_rcp(N2);
        N = N2 * s;
        D = D2 * s;
    }
    return D / N;
}

// I_x(a, b), 1 - I_x(a, b) and the prefactor x^a (1-x)^b / B(a, b); na / nb
// the pairs of the (a, b) and (b, a) branches, 0: as many as it takes.
__device__ inline void beta_inc64(double a, double b, double lnb, int na, int nb, double x,
                                  double *I, double *Ic, double *front) {
    const double e = exp(a * log(x) + b * log1p(-x) - lnb);
    *front = e;
    const bool direct = x * (a + b + 2.0) < a + 1.0;
    const double A = direct ? a : b, B = direct ? b : a, X = direct ? x : 1.0 - x;
    const int pairs = direct ? na : nb;
    const double v = e * (pairs ? beta_cf64_pairs(A, B, X, pairs) : beta_cf64(A, B, X)) / A;
    *I = direct ? v : 1.0 - v;
    *Ic = direct ? 1.0 - v : v;
}

// Solve I_x(a,b) = z for a root in (0, hi0] (hi0 <= 1); Halley steps bracketed
// by [lo, hi] (every evaluation of the increasing I_x shrinks the bracket); a
// step leaving the bracket falls back to bisection, geometric while the
// bracket spans decades.  A Halley step below 1e-4 of the root ends it: the
// next error is the step's cube times a constant that grows with the shapes.  Largest
// over 200,000 draws a shape, of max(root, mean): 6e-11 for sigma / mean of 0.15 to 0.9,
// 1.3e-9 at (400, 583) in its upper tail, 4e-10 at (7500, 22500), 5e-12 at (7.5e7, 2.25e8),
// whose starting values are closer; a row's mean is off by 2e-11 at most.  FP32 losses
// round at 6e-8 (a test for 1e-14 sits in the noise of I_x for one draw in twelve, and
// the 64 lanes of a wavefront waited for the draw that stalled).  Returns false in *ok
// on failure.
__device__ inline double beta_solve64(double a, double b, double lnb, int na, int nb, double z,
                                      double zc, double x, double hi0, int max_iter, bool *ok) {
    const bool lower = z <= zc;
    double lo = 0.0, hi = hi0;
    if (!(x > 0.0 && x < hi)) x = 0.5 * hi;
    *ok = false;
    for (int it = 0; it < max_iter; ++it) {
        double I, Ic, front;
        beta_inc64(a, b, lnb, na, nb, x, &I, &Ic, &front);
        const double r = lower ? (I - z) : (zc - Ic);
        if (r == 0.0) { *ok = true; return x; }
        if (r < 0.0) lo = x; else hi = x;
        // the root lies below 1e-100 (near-Bernoulli shapes): 0, as the FP32
        // loss it scales is
        if (hi <= 1e-100) { *ok = true; return 0.0; }
        const double w = 1.0 - x;
        const double rf = r / front;
        const double uh = rf * fma(a - 1.0, w, -(b - 1.0) * x);
        double xn = x - rf * (x * w) / (1.0 - 0.5 * fmin(1.0, uh));
        const bool halley = xn > lo && xn < hi;
        if (!halley) {
            if (lo > 0.0 && hi > 4.0 * lo) xn = sqrt(lo * hi);
            else if (lo == 0.0) xn = 1e-3 * hi;
            else xn = 0.5 * (lo + hi);
        }
        if ((halley && fabs(xn - x) <= 1e-4 * xn) || hi - lo <= 1e-15 * hi) {
            *ok = true;
            return xn;
        }
        x = xn;
    }
    return x;
}

// FP64 quantile (any shape a, b > 0; lnb = ln B(a, b); na, nb as beta_inc64):
// the smaller side of the root is solved, the other recovered by 1 - y; at
// most max_iter steps.
__device__ __attribute__((noinline)) inline double beta_quantile64(double a, double b, double lnb, int na, int nb, double z,
                                         double zc, int max_iter, bool *ok) {
    double x, hi0;
    bool root_low;
    if (a >= 1.0 && b >= 1.0) {
        // Abramowitz & Stegun 26.2.22 / 26.5.22 (as beta_guess32, in FP64):
        // within a few per cent of the root for shapes of any size; a root
        // near 1/2 may be solved from the other side, so the bracket is whole
        const bool lowz = z < zc;
        const double t = sqrt(-2.0 * log(lowz ? z : zc));
        double y = t - (2.30753 + 0.27061 * t) / (1.0 + t * (0.99229 + 0.04481 * t));
        if (!lowz) y = -y;
        const double lam = (y * y - 3.0) / 6.0;
        const double ra = 1.0 / (2.0 * a - 1.0), rb = 1.0 / (2.0 * b - 1.0);
        const double rh = 0.5 * (ra + rb);
        const double w = y * sqrt(1.0 / rh + lam) * rh - (rb - ra) * (lam + 5.0 / 6.0 - (2.0 / 3.0) * rh);
        const double g = exp(2.0 * w);
        x = a / (a + b * g);
        root_low = x <= 0.5;
        if (!root_low) x = b * g / (a + b * g);
        x = fmin(x, 0.75);
        hi0 = 1.0;
    } else {
        // the leading term of the small-x expansion I_x ~ x^a / (a B(a, b)), at
        // both ends: a root below 1e-100, or that far below 1, is 0 or 1 to the
        // FP32 loss (nearly every draw of a near-Bernoulli shape)
        const double l0 = (log(z * a) + lnb) / a, l1 = (log(zc * b) + lnb) / b;
        if (l0 < -230.0 || l1 < -230.0) {
            *ok = true;
            return l0 < -230.0 ? 0.0 : 1.0;
        }
        double Ih, Ihc, front;
        beta_inc64(a, b, lnb, na, nb, 0.5, &Ih, &Ihc, &front);
        root_low = (z <= zc) ? (z <= Ih) : (zc >= Ihc);
        x = exp(root_low ? l0 : l1);
        // the expansion's next term
        const double A = root_low ? a : b, B = root_low ? b : a;
        const double c = 1.0 + (1.0 - B) * x / (A + 1.0);
        x = c > 0.1 ? x / c : x;
        if (!(x < 0.5)) x = 0.25;
        hi0 = 0.5;
    }
    const double y = beta_solve64(root_low ? a : b, root_low ? b : a, lnb, root_low ? na : nb,
                                  root_low ? nb : na, root_low ? z : zc, root_low ? zc : z, x, hi0,
                                  max_iter, ok);
    if (y == 0.0) *ok = true;    // root below the smallest double
    return root_low ? y : 1.0 - y;
}

// Local coordinate of interpolation point q of a segment.
__device__ inline double seg_node(int q) {
    return 0.5 * cospi((2.0 * q + 1.0) / (2.0 * kSegCoefs));
}

// The value segment seg of a slot interpolates at its point q, in FP64; a slot's
// segments run lower octaves, upper octaves, deviates.
__device__ inline double slot_point(double a, double b, double lnb, int seg, int q) {
    const double t = seg_node(q);
    double z, zc;
    if (seg < 2 * kOctaves) {
        const bool upper = seg >= kOctaves;
        const double p = ldexp(1.5 + t, (upper ? seg - kOctaves : seg) - 24);
        z = upper ? 1.0 - p : p;
        zc = upper ? p : 1.0 - p;
    } else {
        const double v = 0.5 * ((double)(seg - 2 * kOctaves - kDevHalf) + t);
        z = 0.5 * erfc(-v * 0.70710678118654752);
        zc = 0.5 * erfc(v * 0.70710678118654752);
    }
    bool ok;
    return beta_quantile64(a, b, lnb, 0, 0, z, zc, kF64QuantileIters, &ok);
}

// Coefficients in powers of the local coordinate d of the polynomial through the
// values y at the points of a segment (divided differences, then expanded).  Half of
// all draws fall in two segments, so what rounding c0 to FP32 shifts them by would stay
// in the mean over any number of trials: the quadratic coefficient takes it up (the
// mean of d^2 over the segment is 1/12).  The mean quantile of shapes across [1, 32]^2
// is off by 1.6e-10 of it (root mean square; 9.8e-9 with each coefficient rounded by
// itself), the largest error of a draw stays what the interpolation makes it (2.1e-7).
__device__ inline void seg_fit(double *y, float *out) {
    for (int k = 1; k < kSegCoefs; ++k)
        for (int q = kSegCoefs - 1; q >= k; --q)
            y[q] = (y[q] - y[q - 1]) / (seg_node(q) - seg_node(q - k));
    for (int k = kSegCoefs - 2; k >= 0; --k)
        for (int q = k; q < kSegCoefs - 1; ++q) y[q] -= seg_node(k) * y[q + 1];
    for (int q = 0; q < kSegCoefs; ++q) out[q] = (float)y[q];
    out[2] = (float)(y[2] - 12.0 * ((double)out[0] - y[0]));
}

}  // namespace ara
