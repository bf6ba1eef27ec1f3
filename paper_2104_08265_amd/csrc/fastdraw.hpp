// Binomial and normal-approximation counts decided in FP32 wherever FP32 can decide them
// (arXiv:2104.08265 Sec. 4.3.1).  The sampler of fluct.hpp defines every count as an FP64
// computation; these functions return the same count from FP32 estimates of the same
// quantities, or say that the estimates cannot tell (`sure` false): the caller then runs
// the defining computation.  The counts are therefore those of fluct.hpp, bit for bit.
//
// A binomial count is the number of cumulative sums F(0), F(1), ... (in the order of the
// search) that do not exceed the uniform u, so it is certain once u is further from every
// sum than the estimates' error.  What the errors are, with e = 2^-24 (FP32 rounding, one
// unit in the last place of the hardware's functions being 2 e), sums of worst cases:
//  * the weights: the tile kernel takes them from the erf polynomial (erfpoly.hpp, a few
//    1e-16), the definition from the alternating series det_erf, whose cancellation lets it
//    be off by 5.2e-12 at the edges of 4.2-sigma windows (the sum of its terms' rounding
//    bounds; measured at most 1.2e-13).  A weight is half a difference of two, the other
//    axis' weight at most 1 and both together at most 3/2 below p = 1/2: N p is off by
//    kWeightError N = 8e-12 N, and a sum by at most as much;
//  * p: the two weights rounded to FP32, N times one, that times the other, the division by
//    N: 6 e relative; then 17 bits of mantissa, 64 e; together 70 e, which moves a sum by
//    at most 70 e N p pmf(k): 124 e for the inversion (N p pmf <= 1.77 at N = 20, p near
//    1/2), 28 e s to 40 e s (p near 0 to 1/2) for the search from the mode, s = sqrt(N p);
//  * the first probability: inversion exp(N ln(1 - p)), an exponent of at most 13.9 with
//    9.5 e relative error: 134 e of every sum; mode: 12 e;
//  * each step's ratio: inversion 6 e + 2 e (N + 1) / (N - k) (the difference of c1 / (k + 1)
//    and r), weighed by pmf(k) over the steps at most 88 e; mode 10 e, 8 e s, and e j for
//    the j subtractions behind the numerator of the j-th, e s^2 / 2;
//  * one rounding per subtraction from u: at most 15 e, and 100 e for the long searches;
//  * u: 19 of its 53 bits and half a unit of the last: 16 e; the definition's own rounding
//    (its ln(n!) at N = 2^24): 3 e;
//  * N itself: exact below 2^24; above it (inversion only, p is then below 6e-7) up to 30 e in
//    all, where the terms that grow with p are 70 e smaller.
// Together below 380 e + 8e-12 N = 2.27e-5 + 8e-12 N for the inversion, and for the mode
// search 131 e + (36 e + e s / 2) s <= 131 e + 68 e s (s <= 64; near p = 1/2 131 e + 62 e s).
// The margins are 2.5e-5 = 419 e and 2.5e-5 + 4e-6 s = 419 e + 67 e s, each with 8e-12 N.
// Random inputs leave 0.05 to 0.2% of the cells undecided.
#pragma once

#include <cmath>

#include "fluct.hpp"

namespace wct {

WCT_HD float fast_rcp(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_rcpf(x);
#else
  return 1.0f / x;
#endif
}
WCT_HD float fast_exp2(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_exp2f(x);
#else
  return exp2f(x);
#endif
}
WCT_HD float fast_log2(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_logf(x);
#else
  return log2f(x);
#endif
}
WCT_HD float fast_sqrt(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_sqrtf(x);
#else
  return sqrtf(x);
#endif
}

constexpr float kDrawMargin = 2.5e-5f;       // what the sums must keep from u
constexpr float kDrawMarginSigma = 4e-6f; // times sqrt(N p), for the search from the mode
constexpr int kFastSteps = 126;             // inversion steps at most
constexpr int kFastUnrolled = 21;           // the first that is not unrolled (odd)
constexpr int kFastPasses = 512;            // passes of the search from the mode at most
constexpr float kFastMaxMean = 4096.0f;     // means up to which 512 passes hold eight widths
constexpr float kFastMaxN = 16777216.0f;    // 2^24: up to it FP32 holds N and N - k exactly
constexpr float kWeightError = 8e-12f;      // times N: error of N p from the weights

// A cell surely draws 0 when u + N p is below this: 1 - N p is a lower bound of F(0), taken
// with 1e-5 and the weights' error to spare.  Where p may exceed 1/2 the count runs down from N, not up from 0;
// then N p >= 3/2 for three electrons or more, so only rows of one or two are kept out.
WCT_HD float fast_zero_limit(float N) { return N < 3.0f ? -INFINITY : fmaf(N, -kWeightError, 1.0f - 1e-5f); }

// A cell that waits for its batch, in 64 bits.  x: the probability in [0, 1] (its upper two bits
// are then 0) to 17 bits of mantissa, over the row's index in the work item; y: 19 bits of the
// uniform over the cell's offset in the tile.  Weights are below 0 and above 1 where the edges
// round to five sigma (no infinity, no NaN: they stay below 1e11); the definition counts 0 or N
// there: 0 is decided, 1 left to it.
constexpr uint32_t kEntryRow = 255u;
constexpr int kEntryDstBits = 13;
constexpr uint32_t kEntryDst = (1u << kEntryDstBits) - 1u;
WCT_HD uint32_t float_bits(float v) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __float_as_uint(v);
#else
  return __builtin_bit_cast(uint32_t, v);
#endif
}
WCT_HD float bits_float(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __uint_as_float(v);
#else
  return __builtin_bit_cast(float, v);
#endif
}
WCT_HD uint32_t entry_x(float p, uint32_t row) {
  return (((float_bits(fminf(fmaxf(p, 0.0f), 1.0f)) + 32u) << 2) & ~kEntryRow) | row;
}
WCT_HD uint32_t entry_y(uint32_t w, uint32_t dst) { return (w & ~kEntryDst) | dst; }
WCT_HD float entry_p(uint32_t x) { return bits_float((x & ~kEntryRow) >> 2); }
WCT_HD float entry_u(uint32_t y) { return (float)((y & ~kEntryDst) | (1u << (kEntryDstBits - 1))) * 0x1p-32f; }

// The inversion's steps: f(k + 1) = f(k) (c1 / (k + 1) + nr), with v = u - F(k) and its
// smallest modulus so far.
struct FastSearch {
  float f, v, near, c1, nr;
  int k;
  WCT_HD void step(float inv) {
    f *= fmaf(c1, inv, nr);
    v -= f;
    near = fminf(near, fabsf(v));
    k += v >= 0.0f ? 1 : 0;
  }
};
// The first steps with 1 / (k + 1) in the code, two between tests (a table of them costs a
// scalar load's latency every pass).
template <int J>
WCT_HD void fast_steps(FastSearch& t) {
  if constexpr (J < kFastUnrolled) {
    if (any_lane(t.v >= kDrawMargin)) {
      t.step(1.0f / (float)J);
      t.step(1.0f / (float)(J + 1));
      fast_steps<J + 2>(t);
    }
  }
}

// Inversion from 0 (N p < 10).  The lanes of a wave step together until none searches.
WCT_HD bool fast_inversion(float N, float p, float u, int* count) {
  const float mu = N * p;
  const bool fits = (fmaf(N, kWeightError, mu) < (float)kMuSwitch - 1e-4f) & (p < 0.4999f);
  // -ln(1 - p) = 2 atanh(p / (2 - p))
  const float s = p * fast_rcp(2.0f - p), s2 = s * s;
  float poly = 1.0f / 13.0f;
  poly = fmaf(poly, s2, 1.0f / 11.0f);
  poly = fmaf(poly, s2, 1.0f / 9.0f);
  poly = fmaf(poly, s2, 1.0f / 7.0f);
  poly = fmaf(poly, s2, 1.0f / 5.0f);
  poly = fmaf(poly, s2, 1.0f / 3.0f);
  poly = fmaf(poly, s2, 1.0f);
  float f = fast_exp2((N * s) * poly * (float)(-2.0 * kLog2e));
  // f(k+1) = f(k) (r (N - k)) / (k + 1) = f(k) (r (N + 1) / (k + 1) - r)
  const float r = p * fast_rcp(1.0f - p), c1 = fmaf(r, N, r);
  const float v = fits ? u - f : -1.0f;  // u - F(0); undecided cells do not search
  FastSearch t{f, v, fabsf(v), c1, -r, v >= 0.0f ? 1 : 0};
  fast_steps<1>(t);
  for (int j = kFastUnrolled; j <= kFastSteps; ++j) {  // few waves come here
    if (!any_lane(t.v >= kDrawMargin)) break;
    t.step(fast_rcp((float)j));
  }
  *count = t.k;
  // (the loops above end below kDrawMargin: a lane between the two margins is not sure)
  return fits & (t.near >= fmaf(N, kWeightError, kDrawMargin)) & (t.v < 0.0f);
}

// (1 + e) ln(1 + e) - e over e^2, |e| <= 0.1
WCT_HD float fast_dev(float e) {
  float g = -1.0f / 42.0f;
  g = fmaf(g, e, 1.0f / 30.0f);
  g = fmaf(g, e, -1.0f / 20.0f);
  g = fmaf(g, e, 1.0f / 12.0f);
  g = fmaf(g, e, -1.0f / 6.0f);
  return fmaf(g, e, 0.5f);
}
// ln(n!) less Stirling's n ln n - n + ln(2 pi n) / 2, from 1 / n, n >= 10
WCT_HD float fast_stirling(float rn) {
  const float r2 = rn * rn;
  return rn * fmaf(-r2, fmaf(-r2, 1.0f / 1260.0f, 1.0f / 360.0f), 1.0f / 12.0f);
}

// The search from the mode (N p >= 10).  P(mode) by the saddle-point form (Loader, "Fast and
// accurate computation of binomial probabilities", 2000): with
// x = m - N p, ln P = S(N) - S(m) - S(N - m) - [N p h(x / N p) + N q h(-x / N q)]
// - ln(2 pi m (N - m) / N) / 2, h(e) = (1 + e) ln(1 + e) - e, S the Stirling remainder:
// no large terms cancel.
WCT_HD bool fast_chopdown(float N, float p, float u, int* count) {
  const float a = fmaf(N, p, p);  // (N + 1) p
  const float m = floorf(a), fr = a - m, mu = a - p;
  const float werr = N * kWeightError;
  const float tol = fmaf(a, 6e-6f, werr);  // p's error (71 e relative, and the weights') decides the mode's floor
  const bool fits = (fr > tol) & (fr < 1.0f - tol) & (p < 0.4999f) & (mu > (float)kMuSwitch + 1e-4f + werr) &
                    (mu < kFastMaxMean) & (N < kFastMaxN);
  const float nm = N - m, nq = N - mu, q = 1.0f - p, x = p - fr;
  const float rN = fast_rcp(N), rm = fast_rcp(m), rnm = fast_rcp(nm);
  const float e1 = x * fast_rcp(mu), e2 = -x * fast_rcp(nq);
  const float dev = x * (e1 * fast_dev(e1) - e2 * fast_dev(e2));
  const float corr = fast_stirling(rN) - fast_stirling(rm) - fast_stirling(rnm) - dev;
  const float pm = fast_exp2(corr * (float)kLog2e) * fast_sqrt(N * (rm * rnm) * 0.15915494f);
  const float margin = fmaf(kDrawMarginSigma, fast_sqrt(m), kDrawMargin) + werr;
  const float rp = p * fast_rcp(q), rq = q * fast_rcp(p);
  float v = fits ? u - pm : -1.0f;
  float near = fabsf(v), lo = pm, hi = pm;
  float nlo = m * rq, dlo = nm + 1.0f;   // the next step's P ratio below the mode: nlo / dlo
  float nhi = nm * rp, dhi = m + 1.0f;   // above: nhi / dhi
  int c = v >= 0.0f ? 1 : 0;  // intervals (mode, below, above, below, ...) that u lies beyond
  for (int j = 0; j < kFastPasses; ++j) {
    if (!any_lane(v >= margin)) break;
    const float rd = fast_rcp(dlo * dhi);
    lo *= nlo * (rd * dhi);
    hi *= nhi * (rd * dlo);
    nlo = fmaxf(nlo - rq, 0.0f);  // 0 from the last step on: a lane whose search has ended
    nhi = fmaxf(nhi - rp, 0.0f);  // keeps stepping beside the slower ones
    dlo += 1.0f;
    dhi += 1.0f;
    v -= lo;
    near = fminf(near, fabsf(v));
    c += v >= 0.0f ? 1 : 0;
    v -= hi;
    near = fminf(near, fabsf(v));
    c += v >= 0.0f ? 1 : 0;
  }
  *count = (int)m + ((c & 1) ? -((c + 1) >> 1) : (c >> 1));
  return fits & (near >= margin) & (v < 0.0f);
}

// The normal mode's pair: z to within 1.3e-5 (the logarithm loses relative accuracy next to
// u1 = 1, so pairs with u1 > 1 - 2^-10 are left to the defining computation).
WCT_HD bool fast_normal_pair(uint32_t w0, uint32_t w1, uint32_t w2, float* z_even, float* z_odd) {
  const uint32_t a = ~w0 >> 6, b = (1u << 27) - (w1 >> 5);
  const float u1 = fmaf((float)a, 0x1p-26f, (float)b * 0x1p-53f);
  const float r = fast_sqrt(fast_log2(u1) * (float)(-2.0 * kLn2));
  const float f = (float)(w2 & 0x3fffffffu) * 0x1p-30f;
  const bool swap = f > 0.5f;
  const float t = (swap ? 1.0f - f : f) * (float)kHalfPi, t2 = t * t;
  float s = 1.0f / 362880.0f;
  s = fmaf(s, t2, -1.0f / 5040.0f);
  s = fmaf(s, t2, 1.0f / 120.0f);
  s = fmaf(s, t2, -1.0f / 6.0f);
  s = fmaf(s * t2, t, t);
  float c = -1.0f / 3628800.0f;
  c = fmaf(c, t2, 1.0f / 40320.0f);
  c = fmaf(c, t2, -1.0f / 720.0f);
  c = fmaf(c, t2, 1.0f / 24.0f);
  c = fmaf(c, t2, -0.5f);
  c = fmaf(c, t2, 1.0f);
  const float sp = swap ? c : s, cp = swap ? s : c;
  const uint32_t j = w2 >> 30;
  const float ze = (j & 1) ? sp : cp, zo = (j & 1) ? cp : sp;  // up to their signs
  *z_even = r * ((j == 1 || j == 2) ? -ze : ze);
  *z_odd = r * (j >= 2 ? -zo : zo);
  return u1 <= 1.0f - 0x1p-10f;
}

// The normal mode's count: certain unless x = mu + sd z + 1/2 is within its error of a whole
// number (mu: 6 e relative, sd: 14 e, z: 1.3e-5) or reaches the clamp at N.  The weights' error
// of mu, d = kWeightError N, moves sd by d / (2 sd): below sd = 0.05 no |z| <= 8.6 takes x
// away from 1/2 by as much as 0.44, above it x moves by at most d (1 + 8.6 / 0.1) < 100 d.
// sd takes 1 - p: next to p = 1 (windows inside a cell) p's 6 e would be a large part of it, so
// cells from p = 3/4 up are left to the defining computation (sd: 14 e below).
WCT_HD bool fast_normal_count(float N, float mu, float p, float z, int* count) {
  const float sd = fast_sqrt(fmaxf(mu * (1.0f - p), 0.0f));
  const float x = fmaf(sd, z, mu) + 0.5f;
  const float fl = floorf(x), fr = x - fl;
  const float margin = fmaf(sd, 3e-5f, fmaf(mu, 1e-6f, fmaf(N, 100.0f * kWeightError, 2e-6f)));
  *count = (int)fmaxf(fl, 0.0f);
  return (fr > margin) & (fr < 1.0f - margin) & (x < N) & (p < 0.75f);
}

}  // namespace wct
