// dd_device.h -- device math for the damage-diffusion pair term on gfx950.
//
// The pair term of Eqs. 1-4 (Sec. II) in pitch units is
//   phi_hat = E1(x1) - E1(x0),  x1 = a rb1 < x0 = a rb0,  and ln(b1/b0) at a = 0.
// Three evaluation forms are used, chosen by dx = x0 - x1 = a c:
//   * series  (dx <= threshold): exp(-x1) * sum_m P_m dx^m with per-lag P_m
//     (see dd_internal.h); covers a = 0, the small-argument regime and the
//     near-coincident regime without cancellation;
//   * direct  (dx above threshold): E1(x1) - E1(x0) with E1 from its power
//     series (x <= 2.5) or its continued fraction (x > 2.5); the two values
//     differ by more than a factor e^-dx so the subtraction loses < 2 digits;
//   * FP32 series with a split exponent for the mixed-precision bulk.
#pragma once
#include <hip/hip_runtime.h>

#include "dd_internal.h"

namespace dd {

// Load of read-only data through the constant address space: where the
// address is the same for the whole wave (a lag row, a visit position shared
// by all pixels) it becomes a scalar load, also when the pointer itself was
// read from memory (the batched kernels' per-scan descriptors).  Only for
// device-memory tables that no kernel writes while the caller runs: a pointer
// to a thread's private array or to LDS is not a valid constant address, so
// helpers that may receive such rows (phi_general_f64, series_f64_q,
// series_f32_q, as k_pair_terms calls them) read through plain pointers.
#define DD_CONST_AS __attribute__((address_space(4)))
__device__ __forceinline__ float ldc(const float* p) {
  return *reinterpret_cast<const DD_CONST_AS float*>(reinterpret_cast<uintptr_t>(p));
}
__device__ __forceinline__ double ldc(const double* p) {
  return *reinterpret_cast<const DD_CONST_AS double*>(reinterpret_cast<uintptr_t>(p));
}
__device__ __forceinline__ float2 ldc(const float2* p) {
  typedef float v2 __attribute__((ext_vector_type(2)));
  const v2 v = *reinterpret_cast<const DD_CONST_AS v2*>(reinterpret_cast<uintptr_t>(p));
  return make_float2(v[0], v[1]);
}
__device__ __forceinline__ float4 ldc(const float4* p) {
  typedef float v4 __attribute__((ext_vector_type(4)));
  const v4 v = *reinterpret_cast<const DD_CONST_AS v4*>(reinterpret_cast<uintptr_t>(p));
  return make_float4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ double2 ldc(const double2* p) {
  typedef double v2 __attribute__((ext_vector_type(2)));
  const v2 v = *reinterpret_cast<const DD_CONST_AS v2*>(reinterpret_cast<uintptr_t>(p));
  return make_double2(v[0], v[1]);
}
#undef DD_CONST_AS

constexpr double kLog2e = 1.4426950408889634;
constexpr double kLn2 = 0.6931471805599453;
constexpr double kEulerGamma = 0.5772156649015329;

// 1/k! for k = 0 .. 23, each the correctly rounded quotient of two exact
// doubles (k! is exact in double up to 18!; beyond, the first rounding).
struct InvFact {
  double v[24];
  constexpr InvFact() : v() {
    double f = 1.0;
    for (int k = 0; k < 24; ++k) {
      if (k > 0) f *= k;
      v[k] = 1.0 / f;
    }
  }
};

// 2^-y for y >= 0 in double precision, y -> 2^-n 2^-f with n = rint(y),
// f in [-1/2, 1/2]; 2^-f = e^{-f ln 2} by its Taylor polynomial of degree
// DEG: relative remainder < 1.3e-14 for DEG = 11 (the FP64 path's per-term
// budget is 1e-13).
// Returns 0 for y > 1100.
template <int DEG = 11>
__device__ __forceinline__ double exp2_neg(double y) {
  constexpr InvFact f{};
  y = fmin(y, 1100.0);
  const double n = __builtin_rint(y);
  const double g = (n - y) * kLn2;  // e^g with |g| <= 0.3466
  double p = f.v[DEG];
#pragma unroll
  for (int k = DEG - 1; k >= 0; --k) p = fma(p, g, f.v[k]);
  return __builtin_ldexp(p, -(int)n);
}

// cos on [0, pi/2] by its Taylor series (compile time).
constexpr double cheb_cos(double x) {
  double t = 1.0, s = 1.0;
  for (int k = 1; k < 24; ++k) {
    t *= -x * x / ((2.0 * k - 1.0) * (2.0 * k));
    s += t;
  }
  return s;
}
// 2^h for |h| <= 1/2 by the degree-D polynomial interpolating it at the D + 1
// Chebyshev points of that interval (near-minimax), as monomial coefficients
// in h formed at compile time: Chebyshev coefficients by the discrete cosine
// sum over the nodes (T_k(x_j) by the three-term recurrence), then each T_k
// expanded in powers of x = 2h.  Its error is close to the first omitted
// Chebyshev coefficient, 2 I_{D+1}(ln(2) / 2) ~ (ln(2)/4)^{D+1} / (D+1)! 2:
// 1.3e-14 relative at D = 9, the accuracy the degree-11 Taylor polynomial has.
template <int D>
struct Exp2Cheb {
  double c[D + 1];
  constexpr Exp2Cheb() : c() {
    constexpr int N = D + 1;
    constexpr double pi = 3.141592653589793;
    double x[N] = {}, f[N] = {}, a[N] = {};
    for (int j = 0; j < N; ++j) {
      const double th = pi * (j + 0.5) / N;
      // cos on [0, pi/2] only, by symmetry
      x[j] = th <= pi / 2 ? cheb_cos(th) : -cheb_cos(pi - th);
      // 2^{x/2} = e^{x ln2 / 2} by its Taylor series
      const double g = x[j] * 0.34657359027997264;
      double t = 1.0, s = 1.0;
      for (int k = 1; k < 30; ++k) {
        t *= g / k;
        s += t;
      }
      f[j] = s;
    }
    for (int j = 0; j < N; ++j) {
      double tm = 1.0, tk = x[j];
      a[0] += f[j];
      if (N > 1) a[1] += f[j] * tk;
      for (int k = 2; k < N; ++k) {
        const double tn = 2.0 * x[j] * tk - tm;
        tm = tk;
        tk = tn;
        a[k] += f[j] * tk;
      }
    }
    for (int k = 0; k < N; ++k) a[k] *= (k == 0 ? 1.0 : 2.0) / N;
    // monomial coefficients of T_k in x, accumulated with weights a_k
    double tm[N] = {}, tk[N] = {}, px[N] = {};
    tm[0] = 1.0;          // T_0
    if (N > 1) tk[1] = 1.0;  // T_1
    px[0] += a[0];
    if (N > 1) px[1] += a[1];
    for (int k = 2; k < N; ++k) {
      double tn[N] = {};
      for (int m = 0; m < N; ++m) {
        tn[m] = -tm[m] + (m > 0 ? 2.0 * tk[m - 1] : 0.0);
      }
      for (int m = 0; m < N; ++m) {
        tm[m] = tk[m];
        tk[m] = tn[m];
        px[m] += a[k] * tn[m];
      }
    }
    double sc = 1.0;  // x = 2h
    for (int m = 0; m < N; ++m) {
      c[m] = px[m] * sc;
      sc *= 2.0;
    }
  }
};

// 2^-y for y >= 0 to the FP64 series' per-term budget (1e-13): -y -> m + h,
// m = rint(-y), |h| <= 1/2, 2^h by Exp2Cheb<9> (relative error below 1.9e-14,
// two FMAs fewer than the degree-11 Taylor form of exp2_neg); rounding -y
// rather than y gives the exponent without a negation.  Returns 0 for
// y > 1100.
__device__ __forceinline__ double exp2_neg9(double y) {
  constexpr Exp2Cheb<9> e{};
  const double ny = -fmin(y, 1100.0);
  const double m = __builtin_rint(ny);
  const double h = ny - m;
  double p = e.c[9];
#pragma unroll
  for (int k = 8; k >= 0; --k) p = fma(p, h, e.c[k]);
  return __builtin_ldexp(p, (int)m);
}

// Coefficients (-1)^n / (n n!) of the E1 power series, n = 1..24.
struct E1SeriesCoef {
  double c[24];
  constexpr E1SeriesCoef() : c() {
    double fact = 1.0;
    for (int n = 1; n <= 24; ++n) {
      fact *= n;
      c[n - 1] = ((n & 1) ? -1.0 : 1.0) / (n * fact);
    }
  }
};

// E1(x) for x > 0.  Power series about 0 (A&S 5.1.11) for x <= 2.5.  Above:
//   e1_f64: x e^x E1(x) as a polynomial of degree 27 in t = 5/x - 1 on [-1, 1],
//     interpolating it at the Chebyshev points (formed in 50 digits), times e^-x
//     / x: < 3e-15 for x <= 2.5 (24 terms), < 1e-14 above.  It costs a wave the same
//     whatever its lanes' x; the continued fraction, 5 + 90/x levels, took as many
//     as the wave's smallest x (25600 visits of a measured raster list, FP64
//     arrival: 1.21 ms, 1.08 with this).
//   e1_mixed: the even continued fraction
//       E1(x) = e^-x / (x+1 - 1/(x+3 - 4/(x+5 - ...)))   (A&S 5.1.22)
//     to 4 + 30/x levels by the forward three-term recurrence of its convergents,
//     e^-x by degree 7, 18 series terms: < 1e-8.  (A polynomial of degree 16 is
//     quicker by a tenth of a near band and exact to 1e-10, but moves small scans'
//     maps by that 1e-8's share, 2e-9.)
// The polynomials' coefficients are read through the scalar cache where they are
// used: as literals the compiler kept them in vector registers over the whole
// loop, and spilled.
struct E1Coef {
  double e1s[24], e1p[28], exp[12];
};
constexpr E1Coef e1_coef64() {
  E1Coef m{};
  constexpr E1SeriesCoef s{};
  constexpr InvFact f{};
  for (int k = 0; k < 24; ++k) m.e1s[k] = s.c[k];
  for (int k = 0; k < 12; ++k) m.exp[k] = f.v[k];
  constexpr double p[28] = {
      0.85211088142366054,     -0.11266528854196572,    0.024605713456218568,
      -0.0069088524922641479,  0.0022722723724399197,   -0.00083528067421447471,
      0.00033385513528776421,  -0.00014252919697465435, 6.4195520285397357e-05,
      -3.0236875189450238e-05, 1.4826575324334165e-05,  -7.5024747375011427e-06,
      3.7373281248863727e-06,  -1.9692852600550294e-06, 1.6580230589741762e-06,
      -9.9746100573012787e-07, -8.5413108906820068e-07, 6.3860956694177865e-07,
      2.0636461768882854e-06,  -1.4255097338348177e-06, -2.0772284268090886e-06,
      1.4497712328551951e-06,  1.5337473362622037e-06,  -1.0651451258185052e-06,
      -6.423368262048952e-07,  4.4610121677846819e-07,  1.3207590773136581e-07,
      -9.1218064392828507e-08};
  for (int k = 0; k < 28; ++k) m.e1p[k] = p[k];
  return m;
}
static __constant__ E1Coef g_e1_coef64 = e1_coef64();

// The series' part, NS terms.
template <int NS, typename C>
__device__ __forceinline__ double e1_series(double x, const C* c) {
  double s = ldc(c->e1s + NS - 1);
#pragma unroll
  for (int n = NS - 2; n >= 0; --n) s = fma(s, x, ldc(c->e1s + n));
  return -kEulerGamma - ::log(x) - x * s;
}
// e^-x as in exp2_neg, degree NE.
template <int NE, typename C>
__device__ __forceinline__ double e1_exp(double x, const C* c) {
  const double y = fmin(x * kLog2e, 1100.0), n = __builtin_rint(y), g = (n - y) * kLn2;
  double e = ldc(c->exp + NE);
#pragma unroll
  for (int k = NE - 1; k >= 0; --k) e = fma(e, g, ldc(c->exp + k));
  return __builtin_ldexp(e, -(int)n);
}

__device__ __forceinline__ double e1_f64(double x) {
  const E1Coef* c = &g_e1_coef64;
  asm volatile("" : "+s"(c));  // loads through it stay behind this point
  if (x <= 2.5) return e1_series<24>(x, c);
  double r = __builtin_amdgcn_rcp(x);  // 1/x, by two Newton steps
  r = fma(fma(-x, r, 1.0), r, r);
  r = fma(fma(-x, r, 1.0), r, r);
  const double t = fma(5.0, r, -1.0);
  double p = ldc(c->e1p + 27);
#pragma unroll
  for (int k = 26; k >= 0; --k) p = fma(p, t, ldc(c->e1p + k));
  return e1_exp<11>(x, c) * (p * r);
}

struct MixedCoef {
  double e1s[18], exp[8];
};
constexpr MixedCoef mixed_coef() {
  MixedCoef m{};
  constexpr E1SeriesCoef s{};
  constexpr InvFact f{};
  for (int k = 0; k < 18; ++k) m.e1s[k] = s.c[k];
  for (int k = 0; k < 8; ++k) m.exp[k] = f.v[k];
  return m;
}
static __constant__ MixedCoef g_mixed_coef = mixed_coef();
__device__ __forceinline__ const MixedCoef* mixed_coef_here() {
  const MixedCoef* c = &g_mixed_coef;
  asm volatile("" : "+s"(c));  // loads through it stay behind this point
  return c;
}

__device__ __forceinline__ double e1_mixed(double x, const MixedCoef* c) {
  if (x <= 2.5) return e1_series<18>(x, c);
  const int depth = 4 + (int)(30.0 / x);
  double am1 = 1.0, bm1 = 0.0, a0 = x + 1.0, b0 = 1.0;
  double bj = x + 1.0;
  for (int j = 1; j <= depth; ++j) {
    bj += 2.0;
    const double aj = -(double)j * (double)j;
    const double a1 = fma(bj, a0, aj * am1);
    const double b1 = fma(bj, b0, aj * bm1);
    am1 = a0; bm1 = b0; a0 = a1; b0 = b1;
  }
  return e1_exp<7>(x, c) * (b0 / a0);
}

// Series form in double precision with P_0..P_M read from an FP64 row.
// The two factors of the term: returns q and sets t = exp(-x1) (term = t q).
template <int M>
__device__ __forceinline__ double series_f64_q(double a, const double* __restrict__ row,
                                               double& t) {
  const double z = a * row[kR64_C];
  double q = row[kR64_P + M];
#pragma unroll
  for (int m = M - 1; m >= 0; --m) q = fma(q, z, row[kR64_P + m]);
  t = exp2_neg9(a * row[kR64_RL2]);
  return q;
}

template <int M>
__device__ __forceinline__ double series_f64(double a, const double* __restrict__ row) {
  double t;
  const double q = series_f64_q<M>(a, row, t);
  return t * q;
}

// General FP64 pair term: series for dx <= 1, direct difference above.
__device__ __forceinline__ double phi_general_f64(double a, const double* __restrict__ row) {
  const double z = a * row[kR64_C];
  if (z <= kThr64) return series_f64<kM64>(a, row);
  const double x1 = a * row[kR64_RB1];
  if (x1 > 745.0) return 0.0;  // both E1 values below the double range
  const double x0 = a * row[kR64_RB0];
  const double e0 = x0 > 745.0 ? 0.0 : e1_f64(x0);
  return e1_f64(x1) - e0;
}

// General pair term of the mixed path, for the pairs its FP32 series does not
// cover (dx > 0.25), to ~1e-8 relative, a hundredth of the mixed bound:
// dx <= 1: the series of degree 12 (truncation < 2e-9) in FP64 times
// exp(-x1) in the split FP32 form of the bulk (a exact, x1 log2(e) = yh + yl);
// dx > 1: E1(x1) - E1(x0) by e1_mixed (the two values differ by more than a
// factor e, so the difference keeps ~2e-8).
__device__ __forceinline__ double phi_general_mixed(float a, const double* __restrict__ r64,
                                                    const float* __restrict__ r32,
                                                    const MixedCoef* c) {
  const double ad = (double)a;
  const double z = ad * r64[kR64_C];
  if (z <= kThr64) {
    double q = r64[kR64_P + 12];
#pragma unroll
    for (int m = 11; m >= 0; --m) q = fma(q, z, r64[kR64_P + m]);
    const float rhi = r32[kR32_RHI];
    const float yh = a * rhi;
    float yl = __builtin_fmaf(a, rhi, -yh);
    yl = __builtin_fmaf(a, r32[kR32_RLO], yl);
    float t = __builtin_amdgcn_exp2f(-yh);
    t = __builtin_fmaf(t, yl * (float)(-kLn2), t);
    return (double)t * q;
  }
  const double x1 = ad * r64[kR64_RB1];
  if (x1 > 745.0) return 0.0;
  const double x0 = ad * r64[kR64_RB0];
  const double e0 = x0 > 745.0 ? 0.0 : e1_mixed(x0, c);
  return e1_mixed(x1, c) - e0;
}

// Its series part, 0.25 < dx <= kMidDx, with the rows read as uniform.
constexpr float kMidDx = (float)kThr64;
__device__ __forceinline__ double phi_mid_mixed(float a, const double* __restrict__ r64,
                                                const float* __restrict__ r32) {
  const double z = (double)a * ldc(r64 + kR64_C);
  double q = ldc(r64 + kR64_P + 12);
#pragma unroll
  for (int m = 11; m >= 0; --m) q = fma(q, z, ldc(r64 + kR64_P + m));
  const float rhi = ldc(r32 + kR32_RHI);
  const float yh = a * rhi;
  float yl = __builtin_fmaf(a, rhi, -yh);
  yl = __builtin_fmaf(a, ldc(r32 + kR32_RLO), yl);
  float t = __builtin_amdgcn_exp2f(-yh);
  t = __builtin_fmaf(t, yl * (float)(-kLn2), t);
  return (double)t * q;
}

// Mixed-precision series with P_0..P_M from an FP32 row.  `a` is exact
// (lattice distances).  x1 log2(e) = a (rhi + rlo) is formed as yh + yl with
// yh = fl(a rhi) and yl its rounding error plus a rlo, so that
// exp(-x1) = 2^-yh (1 - ln2 yl) keeps its relative error near 1e-7 even when
// x1 is large.  dx = a c stays below the series threshold, where the sum is
// well conditioned.
// The two factors of the term: returns q and sets t = 2^-yh (term = t q).
template <int M>
__device__ __forceinline__ float series_f32_q(float a, const float* __restrict__ row, float& t) {
  const float z = a * row[kR32_C];
  const float rhi = row[kR32_RHI];
  const float yh = a * rhi;
  float yl = __builtin_fmaf(a, rhi, -yh);
  yl = __builtin_fmaf(a, row[kR32_RLO], yl);
  t = __builtin_amdgcn_exp2f(-yh);
  float q;
  if constexpr (M == 0) {
    q = row[kR32_P0];
  } else {
    q = row[kR32_P1 + M - 1];
#pragma unroll
    for (int m = M - 1; m >= 1; --m) q = __builtin_fmaf(q, z, row[kR32_P1 + m - 1]);
    q = __builtin_fmaf(q, z, row[kR32_P0]);
  }
  return __builtin_fmaf(q, yl * (float)(-kLn2), q);
}

template <int M>
__device__ __forceinline__ float series_f32(float a, const float* __restrict__ row) {
  float t;
  const float q = series_f32_q<M>(a, row, t);
  return t * q;
}

// Mixed-precision series for degree M <= 3 in powers of a itself,
//   q = P_0 + PA_1 a + ... + PA_M a^M,   PA_m = P_m c^m,
// with the exponent's rounding correction folded in: with x1 log2(e) =
// yh + e2 + a rlo (yh = fl(a rhi), e2 its exact rounding error),
// exp(-x1) = 2^-yh (1 + eps), eps = -ln2 (e2 + a rlo), and
// t q (1 + eps) ~= t (q + P_0 eps); the neglected t P_0 eps (q/P_0 - 1) is
// below |eps| dx / 2, i.e. under 1e-8 of the term at the dx <= 0.01 where
// degrees <= 3 are used.  P_0 eps enters as -ln2 P_0 rlo added to the linear
// coefficient (row field PA_1 holds PA_1 - ln2 P_0 rlo) and one fma with e2.
// `a` is exact.  COMP = false leaves out the e2 correction, for rows where
// y = x1 log2(e) is small enough that fl(a rhi) alone is accurate enough.
template <int M, bool COMP = true>
__device__ __forceinline__ float series_f32a_q(float a, const RowA& w, float& t) {
  static_assert(M <= kMaxA, "degree too high for the a-form");
  const float yh = a * w.rhi;
  t = __builtin_amdgcn_exp2f(-yh);
  float q;
  if constexpr (M == 0) {
    q = __builtin_fmaf(w.p0nr, a, w.p0);
  } else {
    const float pa[3] = {w.pa1, w.pa2, w.pa3};
    q = pa[M - 1];
#pragma unroll
    for (int m = M - 1; m >= 1; --m) q = __builtin_fmaf(q, a, pa[m - 1]);
    q = __builtin_fmaf(q, a, w.p0);
  }
  if constexpr (!COMP) return q;
  const float e2 = __builtin_fmaf(a, w.rhi, -yh);
  return __builtin_fmaf(w.p0n, e2, q);
}

template <int M, bool COMP = true>
__device__ __forceinline__ float series_f32a(float a, const RowA& w) {
  float t;
  const float q = series_f32a_q<M, COMP>(a, w, t);
  return t * q;
}

// Marks a non-finite output value in the word of `f` (see OutFlag).
__device__ __forceinline__ void flag_nonfinite(const OutFlag& f, double v, int64_t idx) {
  if (__builtin_isfinite(v) || f.word == nullptr) return;
  constexpr unsigned long long lim = (1ull << kFlagIndexBits) - 1;
  unsigned long long i = (unsigned long long)(f.base + idx);
  if (i >= lim) i = lim - 1;
  atomicMax(f.word, (f.seq << kFlagIndexBits) | (lim - i));
}

// The 8 bulk fields of a uniform FP32 row (scalar loads).
__device__ __forceinline__ RowA load_rowa(const float* __restrict__ row) {
  const float4 u = ldc(reinterpret_cast<const float4*>(row));
  const float4 v = ldc(reinterpret_cast<const float4*>(row + 4));
  return RowA{u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
}

}  // namespace dd
