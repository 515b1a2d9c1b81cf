// Element-wise mathematics of the learnable modulation and the softened
// ternarisation (Sec. 2.2-2.3, Eq. 2-6), shared by the LM+ST kernels and by
// the weight-gradient GEMM's fused factor-gradient epilogue.
#pragma once

#include <cmath>

#include "kernels.h"

namespace catq {

// Constants of f at sharpness s (StConst), formed on the host in double.
static inline StConst make_st(double s) {
  StConst c;
  const double l2e = 1.4426950408889634;
  c.c2s = (float)(2.0 * s * l2e);
  c.s4 = (float)(4.0 * s);
  c.s4l = (float)(4.0 * s * l2e);
  c.k2 = (float)(1.0 / std::tanh(s));
  c.sk4 = (float)(2.0 * s / std::tanh(s));
  return c;
}

// 1 - exp(-t) for t >= 0 without cancellation: a degree-7 Taylor polynomial
// below t = 1/4 (truncation < 2e-9 relative), the exponential above it.
__device__ __forceinline__ float one_minus_exp_neg(float t, float t_log2e) {
  if (t < 0.25f) {
    float p = 1.0f / 5040.0f;
    p = fmaf(p, t, -1.0f / 720.0f);
    p = fmaf(p, t, 1.0f / 120.0f);
    p = fmaf(p, t, -1.0f / 24.0f);
    p = fmaf(p, t, 1.0f / 6.0f);
    p = fmaf(p, t, -0.5f);
    p = fmaf(p, t, 1.0f);
    return t * p;
  }
  return 1.0f - __builtin_amdgcn_exp2f(-t_log2e);
}

// Per-group scalars of Eq. 3-4 from fp32 stats and factors.  mu and alpha are
// formed in double (the products of two fp32 values are exact there) and
// rounded once to fp32; Delta likewise.
struct GroupScalars {
  float mu, alpha, alpha_div, delta;
};

__device__ __forceinline__ GroupScalars group_scalars(float mu0, float alpha0, float dmu, float dal,
                                                      float dde, float delta0) {
  GroupScalars g;
  g.mu = (float)((double)mu0 + (double)dmu * (double)alpha0);
  g.alpha = (float)((double)dal * (double)alpha0);
  g.delta = (float)((double)dde * (double)delta0);
  g.alpha_div = fmaxf(g.alpha, 1.17549435e-38f);  // smallest normal: constant groups stay finite
  if (g.alpha != g.alpha) g.alpha_div = g.alpha;  // keep NaN
  return g;
}

// Exact hard decision of Eq. 2 on W_hat = (w - mu)/alpha against Delta,
// without dividing: compare r = w - mu with theta = Delta*alpha in double.
__device__ __forceinline__ float hard_code(float w, float mu, double theta) {
  double r = (double)w - (double)mu;
  return (float)((r > theta) - (r < -theta));
}

// The same decision with a float32 screen.  With r = w - mu and
// theta = Delta*alpha exact, r32 = fl(r) and b = fl(Delta*alpha) each carry a
// relative error of at most 2^-24 (a difference of floats that falls below
// the normal range is exact), so |r32| > b (1 + 2^-21) proves |r| > theta
// and |r32| < b (1 - 2^-21) proves |r| < theta; only the band between them,
// and thresholds outside [2^-120, 2^120] (zero, negative, NaN, huge), go to
// the exact float64 comparison.
struct HardThresh {
  double theta;
  float hi, lo;
};
__device__ __forceinline__ HardThresh hard_thresh(float delta, float alpha_div) {
  HardThresh t;
  t.theta = (double)delta * (double)alpha_div;
  const float b = delta * alpha_div;
  const bool ok = b >= 0x1p-120f && b <= 0x1p+120f;  // false for NaN
  t.hi = ok ? b * (1.0f + 0x1p-21f) : __builtin_inff();
  t.lo = ok ? b * (1.0f - 0x1p-21f) : -1.0f;
  return t;
}
// Codes of N weights of one group: the screen for all N, and the exact
// comparison for all N when any of them falls in the band (rare; one branch).
template <int N>
__device__ __forceinline__ void hard_codes_n(const float (&w)[N], float mu, const HardThresh& t,
                                             float (&c)[N]) {
  bool band = false;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const float r = w[j] - mu;
    const float a = fabsf(r);
    c[j] = a > t.hi ? copysignf(1.0f, r) : 0.0f;
    band |= !(a > t.hi) && !(a < t.lo);
  }
  if (band) {
#pragma unroll
    for (int j = 0; j < N; ++j) c[j] = hard_code(w[j], mu, t.theta);
  }
}
__device__ __forceinline__ void hard_codes8(const float (&w)[8], float mu, const HardThresh& t,
                                            float (&c)[8]) {
  hard_codes_n<8>(w, mu, t, c);
}

// The softened ternarisation of one group in the base-2 exponent domain.
// With z = (w - mu) * sc = 2 s W_hat log2(e), y = |z| and x = |W_hat|:
//   q_a = e^{-2 s |x - Delta|} = 2^{-|y - dz|},   e^{-4 s x} = 2^{-2 y},
//   E = 1 - e^{-4 s x},  q_b = q_a (1 - E) (x < Delta) or q_a (1 - E_Delta),
//   alpha f = copysign(num / ((1 + q_a)(1 + q_b)), z) * alpha / tanh(s),
//   num = E (x >= Delta) or q_a E (x < Delta)
// (the cancellation-free form of Eq. 5; the scalings of the exponents and of
// the output are folded into per-group constants).
struct SoftGroup {
  float mu;     // mu of Eq. 3
  float sc;     // 2 s log2(e) / alpha:  z = (w - mu) * sc
  float inv_a;  // 1 / alpha  (when sc does not fit a float)
  float c2s;    // 2 s log2(e)
  float dz;     // 2 s Delta log2(e)
  float ed;     // E_Delta = 1 - e^{-4 s Delta}
  float ak;     // alpha / tanh(s)
  bool fast;    // sc finite: z in one product
};

__device__ __forceinline__ SoftGroup soft_group(const GroupScalars& gs, const StConst& c) {
  SoftGroup q;
  q.mu = gs.mu;
  q.inv_a = __builtin_amdgcn_rcpf(gs.alpha_div);  // 1 ulp; W_hat needs no more
  q.c2s = c.c2s;
  q.sc = q.inv_a * c.c2s;
  q.fast = fabsf(q.sc) <= 3.0e38f;  // false for inf and NaN
  q.dz = gs.delta * c.c2s;
  q.ed = one_minus_exp_neg(gs.delta * c.s4, gs.delta * c.s4l);
  q.ak = gs.alpha * c.k2;
  return q;
}

// 1 - 2^{-2y} (= 1 - e^{-t}, t = 2 y ln 2) for y >= 0 given T = 2^{-2y}:
// below t = 1/8 the series of 1 - e^{-t} to t^5 in powers of y (truncation
// below 5e-8 relative), above it 1 - T (no cancellation: T < 0.89).
constexpr float kSeriesY = 0.09016844f;
__device__ __forceinline__ float one_minus_exp2_neg2(float y, float T) {
  if (y < kSeriesY) {
    float p = 0.04266738519f;
    p = fmaf(p, y, -0.1538900584f);
    p = fmaf(p, y, 0.4440328777f);
    p = fmaf(p, y, -0.9609060287f);
    p = fmaf(p, y, 1.386294365f);
    return y * p;
  }
  return 1.0f - T;
}

// alpha * f(W_hat; s, Delta) of two weights (Eq. 5 times the group scale).
// The series of E only where some lane of the wave has a small y; the value
// does not depend on that branch.  One branch per two weights: per weight, as the
// compiler places it, the pass over 352M bf16 weights with cached statistics takes
// 276 us, per two 269 us, per eight 282 us.
template <bool FAST>
__device__ __forceinline__ void soft_pair(const float* w, const SoftGroup& q, float* out) {
  float z[2], E[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    z[j] = FAST ? (w[j] - q.mu) * q.sc : ((w[j] - q.mu) * q.inv_a) * q.c2s;
    const float y = fabsf(z[j]);
    E[j] = 1.0f - __builtin_amdgcn_exp2f(-(y + y));
  }
  if (__any(fminf(fabsf(z[0]), fabsf(z[1])) < kSeriesY)) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float y = fabsf(z[j]);
      E[j] = y < kSeriesY ? one_minus_exp2_neg2(y, 0.0f) : E[j];
    }
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const float d = fabsf(z[j]) - q.dz;
    const float qa = __builtin_amdgcn_exp2f(-fabsf(d));
    const bool ge = d >= 0.0f;
    const float eb = ge ? q.ed : E[j];
    const float qb = fmaf(-qa, eb, qa);
    const float opa = 1.0f + qa;
    const float den = fmaf(opa, qb, opa);
    const float num = ge ? E[j] : qa * E[j];
    out[j] = copysignf(num * __builtin_amdgcn_rcpf(den), z[j]) * q.ak;
  }
}

template <int N>
__device__ __forceinline__ void soft_values(const float (&w)[N], const SoftGroup& q,
                                            float (&out)[N]) {
  static_assert(N % 2 == 0, "pairs");
  if (q.fast) {
#pragma unroll
    for (int j = 0; j < N; j += 2) soft_pair<true>(w + j, q, out + j);
  } else {
#pragma unroll
    for (int j = 0; j < N; j += 2) soft_pair<false>(w + j, q, out + j);
  }
}

// The transition function and its derivatives in the backward.  With
// z = 2 s log2(e) W_hat, t = 2^{-|z|} = e^{-2 s |W_hat|} and dz = 2 s log2(e) Delta,
//   E = 1 - t^2,  D = 1 + 2 cosh(2 s Delta) t + t^2,
//   f       = copysign(E / D, z) / tanh(s)
//   f_W     = (2 s / tanh s) t (2 cosh(2 s Delta) (1 + t^2) + 4 t) / D^2
//   f_Delta = -copysign((2 s / tanh s) 2 sinh(2 s Delta) t E / D^2, z)
// (sinh(2u) / (cosh 2u + cosh 2d) = tanh(u - d) / 2 + tanh(u + d) / 2, and its
// derivatives): sums of positive terms only, so no cancellation, and one
// exponential and one reciprocal per weight.  The vector ALU is what bounds
// the factor-gradient epilogue (the form with exponentials of -|x - Delta| and
// -2x and selects at |x| = Delta took ~16 more issue slots per weight).
// 2 sinh is applied to a lane's sum of f_Delta, whose terms are 2^-dz of its
// size until then, and 2^{-|z|} of weights past the threshold must not fall below
// the normal range while it still counts: beyond dz = 60 (the paper's schedule ends
// at dz = 43.3 for d_Delta = 1) a group takes the general form below.  At 60 the
// terms keep all their digits for gradients G from 2^-64 (5e-20) up, and the
// weights that lose some have f_W and f_Delta below 2^-66 of their peak.
// (2 sinh per weight instead, without that limit on G: the routed experts'
// launches 3-8% slower, by another register or a longer chain in the loop.)
constexpr float kFastDz = 60.0f;

// 2 cosh(2 s Delta) and 2 sinh(2 s Delta) (ed = 1 - e^{-4 s Delta}); the
// exponent is formed in float64, so that its rounding (2^-24 of ~50) does not
// enter f, whose dead zone is proportional to 1 / cosh.
struct TransGroup {
  float dz, ed, c2, s2;
  bool fast;
};
__device__ __forceinline__ TransGroup trans_group(float delta, const StConst& c) {
  TransGroup q;
  const double e = (double)delta * (double)c.c2s, n = rint(e);
  q.dz = (float)e;
  q.ed = one_minus_exp_neg(delta * c.s4, delta * c.s4l);
  q.fast = fabsf(q.dz) <= kFastDz;  // false for NaN
  const float p = ldexpf(__builtin_amdgcn_exp2f((float)(e - n)), q.fast ? (int)n : 0);
  q.c2 = p + __builtin_amdgcn_rcpf(p);
  q.s2 = p * q.ed;
  return q;
}

// t = 2^{-|z|} and E = 1 - t^2 of N weights; the series only where some lane of
// the wave has a small |z| (a branch the compiler would otherwise turn into
// the series for every weight).  The value does not depend on the branch.
template <int N>
__device__ __forceinline__ void exp_parts(const float (&z)[N], float (&t)[N], float (&E)[N]) {
  float ym = fabsf(z[0]);
#pragma unroll
  for (int j = 0; j < N; ++j) {
    t[j] = __builtin_amdgcn_exp2f(-fabsf(z[j]));
    E[j] = fmaf(-t[j], t[j], 1.0f);
    ym = fminf(ym, fabsf(z[j]));
  }
  if (__any(ym < kSeriesY)) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const float y = fabsf(z[j]);
      E[j] = y < kSeriesY ? one_minus_exp2_neg2(y, 0.0f) : E[j];
    }
  }
}

// f, f_W and f_Delta without their constant factors in the general form (q_a,
// q_b, E and num as in the softened ternarisation above):
//   f = k2 * fp,   f_W = sk4 * fwp,   f_Delta = sk4 * fdp.
__device__ __forceinline__ void transition_parts_general(float z, float dz, float ed, float& fp,
                                                         float& fwp, float& fdp) {
  const float y = fabsf(z);
  const float d = y - dz;
  const float qa = __builtin_amdgcn_exp2f(-fabsf(d));
  const float E = one_minus_exp2_neg2(y, __builtin_amdgcn_exp2f(-(y + y)));
  const bool ge = d >= 0.0f;
  const float eb = ge ? ed : E;
  const float qb = fmaf(-qa, eb, qa);
  const float opa = 1.0f + qa, opb = 1.0f + qb;
  const float rden = __builtin_amdgcn_rcpf(opa * opb);
  const float r2 = rden * rden;
  const float num = ge ? E : qa * E;
  fp = copysignf(num * rden, z);
  fwp = fmaf(qa, opb * opb, qb * (opa * opa)) * r2;
  const float om = ge ? E : ed;  // 1 - q_a q_b
  fdp = copysignf((qa * eb) * om * r2, -z);
}

// Running sums of the factor gradients of one group over its weights
// (constant factors left out: FacScale and fac_finish below).
struct FacSums {
  float T, one, W, D;  // sum G f, G f_W, G f_W x, G f_Delta
};

// N weights of a group against their gradients G: z and x of each, the hard
// codes where HARD; STE: f_W = 1, f_Delta = 0 (hard mode only).  x is W_hat times
// a constant, and finite where z overflows (alpha at its lower bound): f_W is 0
// there, and 0 times an infinite z would be NaN.
template <int N, bool HARD, bool STE>
__device__ __forceinline__ void fac_terms(const float (&G)[N], const float (&z)[N],
                                          const float (&x)[N], const TransGroup& q,
                                          const float (&hc)[N], FacSums& s) {
  if constexpr (STE) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      s.T = fmaf(G[j], hc[j], s.T);
      s.one += G[j];
      s.W = fmaf(G[j], x[j], s.W);
    }
  } else if (q.fast) {
    float t[N], E[N];
    exp_parts<N>(z, t, E);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const float u = fmaf(t[j], t[j], 1.0f);
      const float r = __builtin_amdgcn_rcpf(fmaf(q.c2, t[j], u));
      const float F = E[j] * r, tr = t[j] * r;
      // (products in this order stay in range for dz up to kFastDz)
      const float h = fmaf(4.0f, t[j], q.c2 * u);
      const float gf = G[j] * ((h * r) * tr);
      const float Gs = __uint_as_float(__float_as_uint(G[j]) ^ (__float_as_uint(z[j]) & 0x80000000u));
      s.T = HARD ? fmaf(G[j], hc[j], s.T) : fmaf(Gs, F, s.T);
      s.one += gf;
      s.W = fmaf(gf, x[j], s.W);
      s.D = fmaf(Gs, F * tr, s.D);
    }
  } else {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      float fp, fwp, fdp;
      transition_parts_general(z[j], q.dz, q.ed, fp, fwp, fdp);
      const float gf = G[j] * fwp;
      s.T = fmaf(G[j], HARD ? hc[j] : fp, s.T);
      s.one += gf;
      s.W = fmaf(gf, x[j], s.W);
      s.D = fmaf(G[j], fdp, s.D);
    }
  }
}
// A lane's sums to those of the general form (f_Delta's 2 sinh, once per lane).
__device__ __forceinline__ void fac_finish(const TransGroup& q, FacSums& s) {
  if (q.fast) s.D *= -q.s2;
}

// Scales of the per-group sums: f is the hard code (HARD, no scale) or k2 fp;
// f_W is 1 under the straight-through estimator; wz turns a sum of
// G f_W z (z = W_hat c2s, or W_hat straight through) into that of G f_W W_hat.
struct FacScale {
  float f, w, d, wz;
};
__device__ __forceinline__ FacScale fac_scale(int mode, int ste, const StConst& c) {
  FacScale k;
  k.f = (mode == CATQ_SOFT) ? c.k2 : 1.0f;
  k.w = ste ? 1.0f : c.sk4;
  k.d = c.sk4;
  k.wz = ste ? 1.0f : c.sk4 / c.c2s;
  return k;
}

}  // namespace catq
