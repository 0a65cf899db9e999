// dd_items.h -- per-work-item device code of libdd, shared by the per-scan
// kernels (dd_kernels.hip) and the persistent batched kernel (dd_batch.hip).
// One wavefront processes one work item; see dd_kernels.hip for the design.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "dd_device.h"
#include "dd_internal.h"

namespace dd {

// ---------------------------------------------------------------------------
// Lag rows (see dd_internal.h for the series).  J_m(w) by 24-node
// Gauss-Legendre on [0, 1] when w <= 1 (the integrand's pole at u = -1/w is at
// least 1 away), by the forward recurrence J_{m+1} = (1/(m+1) - J_m) / w when
// w > 1 (errors shrink by 1/w per step).
__device__ inline void make_row(double lam, double kappa, double s2, const GLNodes& gl, double* r64,
                         float* r32) {
  if (!(lam > 0.0)) {
    for (int k = 0; k < kRow64; ++k) r64[k] = 0.0;
    for (int k = 0; k < kRow32; ++k) r32[k] = 0.0f;
    return;
  }
  const double db = 4.0 * kappa * fmin(lam, 1.0);
  const double b0 = s2 + 4.0 * kappa * fmax(lam - 1.0, 0.0);
  const double b1 = b0 + db;
  const double w = db / b0;
  const double rb1 = 1.0 / b1, rb0 = 1.0 / b0;
  const double c = db / (b0 * b1);
  double J[kM64 + 1];
  if (w <= 1.0) {
    for (int m = 0; m <= kM64; ++m) J[m] = 0.0;
    for (int k = 0; k < kGL; ++k) {
      const double u = gl.x[k];
      double f = gl.w[k] / (1.0 + w * u);
      for (int m = 0; m <= kM64; ++m) {
        J[m] += f;
        f *= u;
      }
    }
  } else {
    J[0] = log1p(w) / w;
    for (int m = 0; m < kM64; ++m) J[m + 1] = (1.0 / (m + 1) - J[m]) / w;
  }
  double P[kM64 + 1];
  P[0] = log1p(w);
  double inv_fact = 1.0;
  for (int m = 1; m <= kM64; ++m) {
    inv_fact /= m;
    P[m] = ((m & 1) ? -1.0 : 1.0) * w * J[m] * inv_fact;
  }
  const double rl2 = rb1 * kLog2e;
  r64[kR64_RB1] = rb1;
  r64[kR64_RB0] = rb0;
  r64[kR64_C] = c;
  r64[kR64_RL2] = rl2;
  for (int m = 0; m <= kM64; ++m) r64[kR64_P + m] = P[m];
  for (int k = kR64_P + kM64 + 1; k < kRow64; ++k) r64[k] = 0.0;
  const float rhi = (float)rl2;
  const float rlo = (float)(rl2 - (double)rhi);
  r32[kR32_RHI] = rhi;
  r32[kR32_P0] = (float)P[0];
  double cm = 1.0;
  for (int m = 1; m <= kMaxA; ++m) {
    cm *= c;
    r32[kR32_PA + m - 1] = (float)(P[m] * cm + (m == 1 ? -kLn2 * P[0] * (double)rlo : 0.0));
  }
  r32[kR32_P0N] = (float)(-kLn2 * P[0]);
  r32[kR32_P0NR] = (float)(-kLn2 * P[0] * (double)rlo);
  r32[kR32_C] = (float)c;
  r32[kR32_RLO] = rlo;
  for (int m = 1; m <= kM32; ++m) r32[kR32_P1 + m - 1] = (float)P[m];
  for (int k = kR32_P1 + kM32; k < kRow32; ++k) r32[k] = 0.0f;
  r32[kR32_RA] = (float)(kLog2e * (rb1 - c * (P[1] / P[0])));
}


// ---------------------------------------------------------------------------
// Small helpers.
__device__ __forceinline__ void wave_sync() {
  // a wave's LDS operations complete in order: a compiler barrier at
  // wavefront scope orders its writes before other lanes' reads
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A wave's BYTES of the 256-thread block's LDS.
template <int BYTES>
__device__ __forceinline__ char* arr_lds() {
  __shared__ __attribute__((aligned(16))) char lds[4][BYTES];
  return lds[threadIdx.x >> 6];
}

__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// ---------------------------------------------------------------------------
// Arrival query, far region, mixed precision.
//
// Forms of the far series by row range (see DegreeBounds): the full form,
// the a-form without the exponent's rounding correction, and the folded
// single exponential P_0 2^{-a RA}.
enum { kFormFull = 0, kFormPlain = 1, kFormFold = 2 };

// A uniform lag row (map tiles): the 8 bulk fields; degrees above 3 read the row in
// place.
template <int M>
using RowSel = typename std::conditional<(M <= kMaxA), RowA, const float*>::type;

template <int M>
__device__ __forceinline__ RowSel<M> fetch_row(const float* __restrict__ rows, int64_t n) {
  if constexpr (M <= kMaxA)
    return load_rowa(rows + n * kRow32);
  else
    return rows + n * kRow32;
}

template <int M>
__device__ __forceinline__ float series_row32(float a, const RowSel<M>& row) {
  if constexpr (M <= kMaxA)
    return series_f32a<M>(a, row);
  else
    return series_f32<M>(a, row);
}

// The term as its two factors (q returned, t set), for sums that must not
// depend on how the compiler fuses products into additions.
template <int M>
__device__ __forceinline__ float series_row32_q(float a, const RowSel<M>& row, float& t) {
  if constexpr (M <= kMaxA)
    return series_f32a_q<M>(a, row, t);
  else
    return series_f32_q<M>(a, row, t);
}

// The squared distances of a wave's pairs come from the matrix cores.  A visit
// is four halves (PosH), (-2x, -2y, sh, sl) with x^2 + y^2 = 4096 sh + sl, and
//   a = |e|^2 + |p|^2 - 2 e.p = (x_e, y_e, 4096, 1) . (-2x, -2y, sh, sl) + |e|^2
// is a four-term dot product with a start value: v_mfma_f32_4x4x4_16b_f16, 16
// independent 4x4 blocks.  It is exact: coordinates are below 2048, so x, y, -2x
// and -2y (even, below 4096) are half-precision values, sh is at most 2048 and sl
// in [-2048, 2047], and every partial sum is a whole number below 2^24.
//
// Lane l = 4 b + c owns the R visits j = J + R u + t, t < R, u = far_unit(b) + 2 c:
// a block's columns are every other unit of R visits, and two blocks share eight
// units (items with an edge: every unit, u = 4 b + c, see kFarSpace).  Step D takes,
// per t, the four earlier visits i = J + R far_unit(b) + t - D - v, v < 4, of block b
// (the A rows) against the block's four columns c: lane (b, c) gets the pairs of
// lags D + 2 R c + v, four consecutive lags per lane and step.  The lag differs
// between a block's lanes, so the fields of the lag rows that the form needs pass
// through a ring of 128 lags in LDS, one row per lane and 64 lags at a time
// (coalesced, prefetched), and are read back by broadcast; lags outside [lo, hi),
// which the slant adds at both ends, get zero coefficients.  Terms are summed in
// groups of R consecutive lags from lo in FP32, then in FP64; with columns two
// groups apart, the parity of a group is that of the step (R = 4) or of v / R
// (R = 2) in every lane (see far_alone).
//
// Bound: VALU issue, in the folded form a product, the exponential (two
// issues) and a fused multiply-add per pair, and 1/R of a conversion and an FP64
// addition; the matrix cores run beside it.  512x512 in random order: far region
// 8.8 ms with a by three FP32 operations per pair from positions in registers,
// 6.5 ms now, of which the vector ALUs issue for 98% (5.9 instructions per pair).
template <int M, int F>
struct FarRow {
  static constexpr int n = F == kFormFold ? 2 : M <= 1 ? 4 : M <= kMaxA ? 8 : 12;
};
constexpr int kRingLags = 128;
constexpr int kRingBytes = kRingLags * 12 * 4;  // per wave

// The fields of a lag row, in the order the ring holds them.
template <int M, int F>
__device__ __forceinline__ void far_row(const float* __restrict__ row, float (&w)[FarRow<M, F>::n]) {
  if constexpr (F == kFormFold) {
    w[0] = row[kR32_RA];
    w[1] = row[kR32_P0];
  } else {
    w[0] = row[kR32_RHI];
    w[1] = row[kR32_P0];
    if constexpr (M <= 1) {
      w[2] = row[M == 0 ? kR32_P0NR : kR32_PA];
      w[3] = row[kR32_P0N];
    } else if constexpr (M <= kMaxA) {
      w[2] = row[kR32_PA];
      w[3] = row[kR32_P0N];
      w[4] = row[kR32_PA + 1];
      w[5] = row[kR32_PA + 2];
      w[6] = w[7] = 0.0f;
    } else {
      w[2] = row[kR32_C];
      w[3] = row[kR32_RLO];
#pragma unroll
      for (int m = 0; m < kM32; ++m) w[4 + m] = row[kR32_P1 + m];
      w[10] = w[11] = 0.0f;
    }
  }
}

// The term as its two factors (q returned, t set).
template <int M, int F>
__device__ __forceinline__ float far_term_q(float a, const float (&w)[FarRow<M, F>::n], float& t) {
  if constexpr (F == kFormFold) {
    t = __builtin_amdgcn_exp2f(-(a * w[0]));
    return w[1];
  } else if constexpr (M <= 1) {
    return series_f32a_q<M, F == kFormFull>(
        a, RowA{w[0], w[1], w[2], 0.f, 0.f, w[3], w[2], 0.f}, t);
  } else if constexpr (M <= kMaxA) {
    return series_f32a_q<M, F == kFormFull>(
        a, RowA{w[0], w[1], w[2], w[4], w[5], w[3], 0.f, 0.f}, t);
  } else {
    float row[kRow32] = {};
    row[kR32_RHI] = w[0];
    row[kR32_P0] = w[1];
    row[kR32_C] = w[2];
    row[kR32_RLO] = w[3];
#pragma unroll
    for (int m = 0; m < kM32; ++m) row[kR32_P1 + m] = w[4 + m];
    return series_f32_q<M>(a, row, t);
  }
}

typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// Visits p[0] .. p[R - 1] (8-byte alignment); CAS: through the global address
// space, for pointers read from memory.
template <int R, bool CAS>
__device__ __forceinline__ void load_posh(const uint2* p, half4_t (&q)[R]) {
  static_assert(R == 2 || R == 4, "16-byte loads of two visits");
  typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(8)));
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int i = 0; i < R; i += 2) {
    u4 v;
    if constexpr (CAS)
      v = *reinterpret_cast<const __attribute__((address_space(1))) u4*>(
          reinterpret_cast<uintptr_t>(p + i));
    else
      v = *reinterpret_cast<const u4*>(p + i);
    q[i] = __builtin_bit_cast(half4_t, u2{v[0], v[1]});
    q[i + 1] = __builtin_bit_cast(half4_t, u2{v[2], v[3]});
  }
}

// Units of R visits between a block's columns, and its first unit (b: lanes 4 b ..
// 4 b + 3).  Items with an edge add their terms one by one, whatever the parity of a
// group; there every unit is a column, and the slant adds half as many lags to each
// segment, which in a small scan is short: 9x7 visits 69 us with every other unit,
// 61 so.
template <bool EDGE>
constexpr int kFarSpace = EDGE ? 1 : 2;
template <bool EDGE>
__device__ __forceinline__ int far_unit(int b) {
  return EDGE ? 4 * b : 8 * (b >> 1) + (b & 1);
}

// Of a group's first two products one is rounded by itself, the other enters by a
// fused multiply-add: 0 if the first (lag lo + R k), 1 if the second.  Either is
// as accurate, but the lags of a scan repeat the same roundings, and which one it
// is moves the far sums of small scans by some 1e-9 together.  The choice by form,
// visit and parity of k is stated so that the sums do not change with the code
// around them; it is the one of the sums from registers that this form replaced.
template <int M>
constexpr int far_alone(bool odd, int t) {
  return M > kMaxA || (odd && t > 0) ? 1 : 0;
}

template <int M, int R, bool EDGE, bool CAS, int F = kFormFull>
__device__ __forceinline__ void arr_far32(int lo, int hi, const uint2* __restrict__ pos, int64_t J,
                                          const half4_t (&e)[R], const float (&ee)[R],
                                          const float* __restrict__ rows, char* lds,
                                          double (&acc)[R]) {
  constexpr int NF = FarRow<M, F>::n, SP = kFarSpace<EDGE>;
  typedef float vec __attribute__((ext_vector_type(NF == 2 ? 2 : 4)));
  constexpr int NV = NF == 2 ? 1 : NF / 4;
  const int lane = threadIdx.x & 63, c = lane & 3;
  const int64_t Jb = J + R * far_unit<EDGE>(lane >> 2);
  vec* const ring = reinterpret_cast<vec*>(lds);
  const int L0 = lo - 3 * SP * R;  // ring entry of lag n: (n - L0) % 128
  // lane l fetches the row of lag L0 + 64 k + l
  auto fetch = [&](int k, float(&w)[NF]) {
    const int n = L0 + 64 * k + lane;
    far_row<M, F>(rows + (int64_t)max(lo, min(n, hi - 1)) * kRow32, w);
    const bool in = n >= lo && n < hi;
#pragma unroll
    for (int i = 0; i < NF; ++i) w[i] = in ? w[i] : 0.0f;
  };
  auto put = [&](int k, const float(&w)[NF]) {
    vec* r = ring + ((64 * k + lane) & (kRingLags - 1)) * NV;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      vec x;
#pragma unroll
      for (int q = 0; q < NF / NV; ++q) x[q] = w[i * (NF / NV) + q];
      r[i] = x;
    }
  };
  const uint2* pa = pos + (Jb - c - L0);  // step s: four visits before per s
  auto load = [&](int s, half4_t(&q)[R]) { load_posh<R, CAS>(pa - 4 * s, q); };
  const int i0 = (int)(Jb - L0);
  auto step = [&](int s, auto odd_step, const half4_t(&A)[R]) {
    f32x4_t a[R];
#pragma unroll
    for (int t = 0; t < R; ++t)
      a[t] = __builtin_amdgcn_mfma_f32_4x4x4f16(A[t], e[t], f32x4_t{ee[t], ee[t], ee[t], ee[t]}, 0,
                                                0, 0);
    float part[R], q0[R], x0[R];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      // groups of R lags are aligned, so that only they can wrap
      const int at = ((4 * s + SP * R * c + v / R * R) & (kRingLags - 1)) + v % R;
      float w[NF];
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const vec x = ring[at * NV + i];
#pragma unroll
        for (int q = 0; q < NF / NV; ++q) w[i * (NF / NV) + q] = x[q];
      }
#pragma unroll
      for (int t = 0; t < R; ++t) {
        float ex;
        const float q = far_term_q<M, F>(a[t][v], w, ex);
        if (EDGE) {
          const float x = i0 + t - 4 * s - v >= 0 ? q * ex : 0.0f;
          part[t] = v % R == 0 ? x : part[t] + x;
        } else {
          const int own = far_alone<M>(R == 4 ? odd_step() : v / R != 0, t);
          if (v % R == 0) q0[t] = q, x0[t] = ex;
          if (v % R == own) part[t] = q * ex;
          if (own == 1 && v % R == 1) part[t] = __builtin_fmaf(q0[t], x0[t], part[t]);
          if (v % R > own) part[t] = __builtin_fmaf(q, ex, part[t]);
        }
        if (v % R == R - 1) acc[t] += (double)part[t];
      }
    }
  };
  wave_sync();  // the ring's last readers are done
  {
    float w0[NF], w1[NF];
    fetch(0, w0);
    fetch(1, w1);
    put(0, w0);
    put(1, w1);
  }
  wave_sync();
  const int steps = (hi - L0 + 3) / 4;
  half4_t A[R], B[R];
  load(0, A);
  load(1, B);
  for (int k = 0; 16 * k < steps; ++k) {
    float w[NF];
    fetch(k + 2, w);
    // an odd count takes one step more, of lags past hi
    const int s1 = min(16 * k + 16, (steps + 1) & ~1);
    for (int s = 16 * k; s < s1; s += 2) {
      step(s, std::false_type{}, A);
      load(s + 2, A);
      step(s + 1, std::true_type{}, B);
      load(s + 3, B);
    }
    wave_sync();
    put(k + 2, w);
    wave_sync();
  }
}

template <int M, int R, bool EDGE>
__device__ __forceinline__ void arr_far64(int lo, int hi, const double2* __restrict__ pos, int64_t jl,
                                          const double (&ex)[R], const double (&ey)[R],
                                          const double* __restrict__ rows, double (&acc)[R]) {
  double2 W[2 * R - 1];
#pragma unroll
  for (int q = 0; q < 2 * R - 1; ++q) W[q] = pos[jl - lo - (R - 1) + q];
  for (int n0 = lo; n0 < hi; n0 += R) {
#pragma unroll
    for (int s = 0; s < R; ++s) {
      const double* row = rows + (int64_t)(n0 + s) * kRow64;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double2 p = W[r - s + R - 1];
        const double dx = ex[r] - p.x, dy = ey[r] - p.y;
        const double a = fma(dy, dy, dx * dx);
        double v = series_f64<M>(a, row);
        if (EDGE) v = (jl + r >= (int64_t)(n0 + s)) ? v : 0.0;
        acc[r] += v;
      }
    }
#pragma unroll
    for (int q = 2 * R - 2; q >= R; --q) W[q] = W[q - R];
    const int64_t base = jl - (n0 + R) - (R - 1);
#pragma unroll
    for (int q = 0; q < R; ++q) W[q] = pos[base + q];
  }
}

// Degree dispatch for one segment (uniform branch).  PLAIN: the a-form
// without the exponent's rounding correction (degrees <= 3 only; the planner
// starts that range below degree 4).
template <int R, bool EDGE, bool CAS, bool PLAIN = false>
__device__ __forceinline__ void arr_far32_seg(int M, int lo, int hi, const uint2* __restrict__ pos,
                                              int64_t J, const half4_t (&e)[R], const float (&ee)[R], const float* __restrict__ rows,
                                              char* lds, double (&acc)[R]) {
  if constexpr (PLAIN) {
    switch (M) {
      case 0: arr_far32<0, R, EDGE, CAS, kFormPlain>(lo, hi, pos, J, e, ee, rows, lds, acc); break;
      case 1: arr_far32<1, R, EDGE, CAS, kFormPlain>(lo, hi, pos, J, e, ee, rows, lds, acc); break;
      case 2: arr_far32<2, R, EDGE, CAS, kFormPlain>(lo, hi, pos, J, e, ee, rows, lds, acc); break;
      default: arr_far32<3, R, EDGE, CAS, kFormPlain>(lo, hi, pos, J, e, ee, rows, lds, acc); break;
    }
    return;
  }
  switch (M) {
    case 0: arr_far32<0, R, EDGE, CAS>(lo, hi, pos, J, e, ee, rows, lds, acc); break;
    case 1: arr_far32<1, R, EDGE, CAS>(lo, hi, pos, J, e, ee, rows, lds, acc); break;
    case 2: arr_far32<2, R, EDGE, CAS>(lo, hi, pos, J, e, ee, rows, lds, acc); break;
    case 3: arr_far32<3, R, EDGE, CAS>(lo, hi, pos, J, e, ee, rows, lds, acc); break;
    case 4: arr_far32<4, R, EDGE, CAS>(lo, hi, pos, J, e, ee, rows, lds, acc); break;
    case 5: arr_far32<5, R, EDGE, CAS>(lo, hi, pos, J, e, ee, rows, lds, acc); break;
    default: arr_far32<6, R, EDGE, CAS>(lo, hi, pos, J, e, ee, rows, lds, acc); break;
  }
}

template <int R, bool EDGE>
__device__ __forceinline__ void arr_far64_seg(int M, int lo, int hi, const double2* __restrict__ pos,
                                              int64_t jl, const double (&ex)[R], const double (&ey)[R],
                                              const double* __restrict__ rows, double (&acc)[R]) {
#define DD_CASE(k) \
  case k: arr_far64<k, R, EDGE>(lo, hi, pos, jl, ex, ey, rows, acc); break;
  switch (M) {
    DD_CASE(0) DD_CASE(1) DD_CASE(2) DD_CASE(3) DD_CASE(4) DD_CASE(5) DD_CASE(6) DD_CASE(7)
    DD_CASE(8) DD_CASE(9) DD_CASE(10) DD_CASE(11) DD_CASE(12) DD_CASE(13) DD_CASE(14)
    DD_CASE(15) DD_CASE(16)
    default: arr_far64<17, R, EDGE>(lo, hi, pos, jl, ex, ey, rows, acc); break;
  }
#undef DD_CASE
}

// Segment [lo, hi) of degree M within [n_lo, n_hi): M runs from m_max down.
__device__ __forceinline__ void seg_range(const DegreeBounds& b, int M, int n_lo, int n_hi, int& lo,
                                          int& hi) {
  lo = max(n_lo, b.b[M]);
  hi = (M == 0) ? n_hi : min(n_hi, b.b[M - 1]);
}

// One wavefront processes one arrival work item (far region).  The sums of
// visit j go to partial[slot * pstride + j - pj0]: pstride = V and pj0 = 0
// for a whole-scan query; a visit range keeps only the columns of its tiles.
template <int R, bool CAS, bool EDGE>
__device__ __forceinline__ void arrival_far32(const ArrItem& item, const uint2* __restrict__ pos,
                                              const float* __restrict__ rows, int64_t V,
                                              const DegreeBounds& bnd, double* __restrict__ partial,
                                              int64_t pstride, int64_t pj0, char* lds) {
  const int lane = threadIdx.x & 63;
  const int64_t J = (int64_t)item.tile * (64 * R);
  const int64_t jl = J + R * (far_unit<EDGE>(lane >> 2) + kFarSpace<EDGE> * (lane & 3));
  half4_t e[R];
  float ee[R];
  double acc[R];
  load_posh<R, CAS>(pos + jl, e);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    ee[r] = __builtin_fmaf(4096.0f, (float)e[r][2], (float)e[r][3]);
    e[r] = half4_t{e[r][0] * (_Float16)-0.5f, e[r][1] * (_Float16)-0.5f, (_Float16)4096.0f,
                   (_Float16)1.0f};
    acc[r] = 0.0;
  }
  // rows [n_lo, fold) by degree segment, each split at `plain`; then the
  // folded rows [fold, n_hi) whatever their degree segment
  const int n_fold = max(item.n_lo, min(item.n_hi, bnd.fold));
  for (int M = bnd.m_max; M >= 0; --M) {
    int lo, hi;
    seg_range(bnd, M, item.n_lo, n_fold, lo, hi);
    if (lo >= hi) continue;
    const int mid = max(lo, min(hi, bnd.plain));
    if (lo < mid) arr_far32_seg<R, EDGE, CAS>(M, lo, mid, pos, J, e, ee, rows, lds, acc);
    if (mid < hi) arr_far32_seg<R, EDGE, CAS, true>(M, mid, hi, pos, J, e, ee, rows, lds, acc);
  }
  if (n_fold < item.n_hi)
    arr_far32<0, R, EDGE, CAS, kFormFold>(n_fold, item.n_hi, pos, J, e, ee, rows, lds, acc);
  const int64_t base = (int64_t)(item.slot_flags & kSlotMask) * pstride - pj0;
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (jl + r < V) partial[base + jl + r] = acc[r];
}

template <int R, bool CAS>
__device__ __forceinline__ void do_arrival_far32(const ArrItem& item, const uint2* __restrict__ pos,
                                                 const float* __restrict__ rows, int64_t V,
                                                 const DegreeBounds& bnd,
                                                 double* __restrict__ partial, int64_t pstride,
                                                 int64_t pj0, char* lds) {
  if (item.slot_flags & kItemEdge)
    arrival_far32<R, CAS, true>(item, pos, rows, V, bnd, partial, pstride, pj0, lds);
  else
    arrival_far32<R, CAS, false>(item, pos, rows, V, bnd, partial, pstride, pj0, lds);
}

template <int R>
__device__ __forceinline__ void do_arrival_far64(const ArrItem& item, const double2* __restrict__ pos,
                                                 const double* __restrict__ rows, int64_t V,
                                                 const DegreeBounds& bnd,
                                                 double* __restrict__ partial, int64_t pstride,
                                                 int64_t pj0) {
  const int lane = threadIdx.x & 63;
  const int64_t jl = (int64_t)item.tile * (64 * R) + (int64_t)R * lane;
  double ex[R], ey[R], acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const double2 e = pos[jl + r];
    ex[r] = e.x;
    ey[r] = e.y;
    acc[r] = 0.0;
  }
  const bool edge = (item.slot_flags & kItemEdge) != 0;
  for (int M = bnd.m_max; M >= 0; --M) {
    int lo, hi;
    seg_range(bnd, M, item.n_lo, item.n_hi, lo, hi);
    if (lo >= hi) continue;
    if (edge)
      arr_far64_seg<R, true>(M, lo, hi, pos, jl, ex, ey, rows, acc);
    else
      arr_far64_seg<R, false>(M, lo, hi, pos, jl, ex, ey, rows, acc);
  }
  const int64_t base = (int64_t)(item.slot_flags & kSlotMask) * pstride - pj0;
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (jl + r < V) partial[base + jl + r] = acc[r];
}

// Near band, mixed precision: the pairs that need the general form (series
// variable above the FP32 series' threshold, x1 within the cull) are few and
// scattered over the lanes; evaluated where they occur, the general form runs
// with most lanes idle.  They are queued instead, per lane in LDS (a and the
// lag), and evaluated by the whole wave whenever some lane's queue could
// overflow, and at the end: the queues are packed into one list at offsets
// from a prefix sum of their lengths, lane l evaluates list entries l, l + 64,
// ..., and each lane then adds its own values in the order it queued them
// (deterministic; the general-form terms of a flush enter the FP64 sum after
// the series terms of the same lags).
// Q entries per lane; the values overwrite the packed list.
template <int Q>
struct NearQueue {
  float a[Q][64];
  int32_t n[Q][64];  // lag | (r << 29)
  union {
    struct {
      float a;
      int32_t n;
    } in;
    double v;
  } list[64 * Q];
};

template <int R, int Q>
__device__ __forceinline__ void near_flush(NearQueue<Q>& q, int& cnt,
                                           const double* __restrict__ rows64,
                                           const float* __restrict__ rows32, double (&acc)[R]) {
  static_assert(R <= 4, "the queue entry holds r in two bits");
  const int lane = threadIdx.x & 63;
  const int c = cnt;
  int s = c;  // inclusive prefix sum of the queue lengths over the lanes
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int t = __shfl_up(s, d);
    if (lane >= d) s += t;
  }
  const int base = s - c, total = __shfl(s, 63);
#pragma unroll
  for (int k = 0; k < Q; ++k)
    if (k < c) {
      q.list[base + k].in.a = q.a[k][lane];
      q.list[base + k].in.n = q.n[k][lane] & 0x1fffffff;
    }
  wave_sync();
  const MixedCoef* coef = mixed_coef_here();
  for (int e = lane; e < total; e += 64) {
    const float a = q.list[e].in.a;
    const int64_t n = q.list[e].in.n;
    q.list[e].v = phi_general_mixed(a, rows64 + n * kRow64, rows32 + n * kRow32, coef);
  }
  wave_sync();
#pragma unroll
  for (int k = 0; k < Q; ++k)
    if (k < c) {
      const int r = q.n[k][lane] >> 29 & 3;
      const double v = q.list[base + k].v;
#pragma unroll
      for (int rr = 0; rr < R; ++rr) acc[rr] += (rr == r) ? v : 0.0;  // no indexed registers
    }
  wave_sync();  // the queues and the list are rewritten next
  cnt = 0;
}

constexpr int kNearQ = 12;

// LDS: sizeof(NearQueue<Q>) bytes per wave (mixed).
// Near band: per-pair regime choice, every pair masked by causality.
template <int R, bool MIXED, int Q = kNearQ>
__device__ __forceinline__ void do_arrival_near(const ArrItem& item, const void* __restrict__ pos_v,
                                                const double* __restrict__ rows64,
                                                const float* __restrict__ rows32, int64_t V,
                                                double* __restrict__ partial, int64_t pstride,
                                                int64_t pj0, char* lds) {
  const int lane = threadIdx.x & 63;
  const int64_t jl = (int64_t)item.tile * (64 * R) + (int64_t)R * lane;
  double acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = 0.0;
  if (MIXED) {
    const float2* pos = (const float2*)pos_v;
    float ex[R], ey[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float2 e = pos[jl + r];
      ex[r] = e.x;
      ey[r] = e.y;
    }
    // G lags per step, the next step's positions and row fields in flight; the
    // queue holds a step's pairs beyond the four that leave it as it is
    constexpr int G = 8 / R, NP = G + R - 1;
    static_assert(Q > G * R, "a step's pairs fit the queue");
    NearQueue<Q>& nq = *reinterpret_cast<NearQueue<Q>*>(lds);
    int cnt = 0;
    float2 p[NP];
    float c0[G], h0[G];
    auto fetch = [&](int n) {  // visits jl - n - (G - 1) .. jl - n + R - 1
#pragma unroll
      for (int q = 0; q < NP; ++q) p[q] = pos[jl - n - (G - 1) + q];
#pragma unroll
      for (int s = 0; s < G; ++s) {
        const float* row = rows32 + (int64_t)min(n + s, item.n_hi - 1) * kRow32;
        c0[s] = ldc(row + kR32_C);
        h0[s] = ldc(row + kR32_RHI);
      }
    };
    if (item.n_lo < item.n_hi) fetch(item.n_lo);
    for (int n = item.n_lo; n < item.n_hi; n += G) {
      if (__ballot(cnt > Q - G * R)) near_flush<R>(nq, cnt, rows64, rows32, acc);
      float a[G][R];
      float c1[G], h1[G];
#pragma unroll
      for (int s = 0; s < G; ++s) {
        c1[s] = c0[s];
        h1[s] = h0[s];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const float2 v = p[G - 1 + r - s];
          const float dx = ex[r] - v.x, dy = ey[r] - v.y;
          a[s][r] = __builtin_fmaf(dy, dy, dx * dx);
        }
      }
      if (n + G < item.n_hi) fetch(n + G);
#pragma unroll
      for (int s = 0; s < G; ++s) {
        if (n + s >= item.n_hi) break;
        bool low[R], any = false;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const bool in = jl + r >= n + s && jl + r < V;
          low[r] = in && a[s][r] * c1[s] <= kThr32;
          any = any || low[r];
          if (in && !low[r] && a[s][r] * h1[s] <= kCull32Log2) {
            nq.a[cnt][lane] = a[s][r];
            nq.n[cnt][lane] = (n + s) | (r << 29);
            ++cnt;
          }
        }
        if (__ballot(any)) {
          float w[kRow32];
#pragma unroll
          for (int k = 0; k < kRow32; ++k) w[k] = ldc(rows32 + (int64_t)(n + s) * kRow32 + k);
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const float v = series_f32<kMNear32>(a[s][r], w);
            acc[r] += low[r] ? (double)v : 0.0;
          }
        }
      }
    }
    if (__ballot(cnt > 0)) near_flush<R>(nq, cnt, rows64, rows32, acc);
  } else {
    const double2* pos = (const double2*)pos_v;
    double ex[R], ey[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double2 e = pos[jl + r];
      ex[r] = e.x;
      ey[r] = e.y;
    }
    for (int n = item.n_lo; n < item.n_hi; ++n) {
      const double* r64 = rows64 + (int64_t)n * kRow64;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int64_t i = jl + r - n;
        if (i >= 0 && jl + r < V) {
          const double2 p = pos[i];
          const double dx = ex[r] - p.x, dy = ey[r] - p.y;
          acc[r] += phi_general_f64(fma(dy, dy, dx * dx), r64);
        }
      }
    }
  }
  const int64_t base = (int64_t)(item.slot_flags & kSlotMask) * pstride - pj0;
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (jl + r < V) partial[base + jl + r] = acc[r];
}

// ---------------------------------------------------------------------------
// Map query, mixed precision (FP64 maps: dd_gauss.hip).  Pixel pix = tile * 64 R
// + R lane + r at (X0 + u DX, Y0 + v DY), u = pix % W, v = pix / W, all at the
// item's time; visit v = K - n.  Pixel and probe coordinates are small dyadic
// numbers (other grids run in FP64), and the squared distances come from the
// matrix cores as in arr_far32: the four visits of lags n .. n + 3 are the rows of
// all 16 blocks of v_mfma_f32_4x4x4_16b_f16, the pixels their columns, and a lane
// gets its pixel's distances to the four.  A pixel coordinate has up to 12 bits:
// where it is no half-precision value, a second instruction adds its last bit.
// Lag rows are uniform (scalar loads).
//
// MM: the host has shown that every partial sum, in whatever order, is exact: in
// units of 4^-q (pixels being multiples of 2^-q) below 2^24, although 4096 sh may
// exceed |p|^2 by 2048.  Other grids (33x33 probes and more at 1/64 or 1/32 pitch,
// far negative coordinates) take the distance by three FP32 operations per pair,
// whose partial sums stay at |e|^2 + |p|^2.
//
// Bound: VALU issue (10.4 instructions per pair; all cycles).  512 maps of 128x128
// over a 64x64 raster scan, far items: 5.0 ms with the distance by three FP32
// operations, 4.4 now.
template <int R, bool MM>
struct MapPix {
  half4_t hi[R], lo[R];  // (x, y, 4096, 1), rounded, and what is left of x and y
  bool wide;             // some `lo` of the grid is not zero
  float ee[R];
};
template <int R>
struct MapPix<R, false> {
  float ex[R], ey[R], ee[R];
};

// The visits of lags n .. n + 3 (visits K - n - 3 .. K - n): a lane's row of them,
// or all four, (-2x, -2y, x^2 + y^2), uniform.
template <bool MM>
struct MapVisits {
  half4_t row;
};
template <>
struct MapVisits<false> {
  float4 v[4];
};
struct MapPos {
  const uint2* half;
  const float4* full;
};
template <bool MM>
__device__ __forceinline__ MapVisits<MM> map_visits(const MapPos& pos, int64_t K, int n) {
  MapVisits<MM> m;
  if constexpr (MM) {
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    m.row = __builtin_bit_cast(
        half4_t, *reinterpret_cast<const __attribute__((address_space(1))) u2*>(
                     reinterpret_cast<uintptr_t>(pos.half + (K - n - (int)(threadIdx.x & 3)))));
  } else {
#pragma unroll
    for (int s = 0; s < 4; ++s) m.v[s] = ldc(pos.full + (K - n - s));
  }
  return m;
}

// A lane's four distances; DIFF: by coordinate differences, where not from the
// matrix cores (the near band, which also rounds to the same value above 2^24).
template <int R, bool DIFF = false>
__device__ __forceinline__ f32x4_t map_dist(const MapVisits<true>& vis, const MapPix<R, true>& px,
                                            int r) {
  f32x4_t a = __builtin_amdgcn_mfma_f32_4x4x4f16(
      vis.row, px.hi[r], f32x4_t{px.ee[r], px.ee[r], px.ee[r], px.ee[r]}, 0, 0, 0);
  if (px.wide) a = __builtin_amdgcn_mfma_f32_4x4x4f16(vis.row, px.lo[r], a, 0, 0, 0);
  return a;
}
template <int R, bool DIFF = false>
__device__ __forceinline__ f32x4_t map_dist(const MapVisits<false>& vis, const MapPix<R, false>& px,
                                            int r) {
  f32x4_t a;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const float4 p = vis.v[s];
    if constexpr (DIFF) {
      const float dx = __builtin_fmaf(0.5f, p.x, px.ex[r]), dy = __builtin_fmaf(0.5f, p.y, px.ey[r]);
      a[s] = __builtin_fmaf(dy, dy, dx * dx);
    } else {
      a[s] = __builtin_fmaf(px.ex[r], p.x, __builtin_fmaf(px.ey[r], p.y, px.ee[r] + p.z));
    }
  }
  return a;
}

template <int M, int R, int U, bool MM>
__device__ __forceinline__ void map_far32(int lo, int hi, int64_t K, const MapPos& pos,
                                          const float* __restrict__ rows, const MapPix<R, MM>& px,
                                          double (&acc)[R]) {
  using Row = RowSel<M>;
  int n = lo;
  if (n + U <= hi) {
    Row cur[U];
    MapVisits<MM> pc[U / 4];
#pragma unroll
    for (int s = 0; s < U; ++s) {
      cur[s] = fetch_row<M>(rows, n + s);
      if (s % 4 == 0) pc[s / 4] = map_visits<MM>(pos, K, n + s);
    }
    for (; n + U <= hi; n += U) {
      Row nxt[U];
      MapVisits<MM> pn[U / 4];
#pragma unroll
      for (int s = 0; s < U; ++s) {
        nxt[s] = fetch_row<M>(rows, min(n + U + s, hi - 1));
        if (s % 4 == 0) pn[s / 4] = map_visits<MM>(pos, K, n + U + s);
      }
      // Groups of four lags in lag order, each summed by an explicit chain
      // of fused multiply-adds: the arithmetic of a pixel is then the same
      // for every tile width and unroll depth.
#pragma unroll
      for (int q = 0; q < U; q += 4) {
        f32x4_t a[R];
#pragma unroll
        for (int r = 0; r < R; ++r) a[r] = map_dist<R>(pc[q / 4], px, r);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          float g = 0.0f;
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            float t;
            const float qv = series_row32_q<M>(a[r][s], cur[q + s], t);
            g = s == 0 ? t * qv : __builtin_fmaf(t, qv, g);
          }
          acc[r] += (double)g;
        }
      }
#pragma unroll
      for (int s = 0; s < U; ++s) cur[s] = nxt[s];
#pragma unroll
      for (int s = 0; s < U / 4; ++s) pc[s] = pn[s];
    }
  }
  for (; n < hi; ++n) {
    const MapVisits<MM> p = map_visits<MM>(pos, K, n);
    const Row row = fetch_row<M>(rows, n);
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] += (double)series_row32<M>(map_dist<R>(p, px, r)[0], row);
  }
}

// One-pixel tiles, degrees <= 3.  A one-pixel tile has too little work per
// lag to hide per-lag scalar loads of rows that are read once (as for a
// single map row), so the rows and probe positions of 64 lags at a time are
// brought into LDS by one vector load per lane, the next 64 in flight while
// the current ones are evaluated, and read back by broadcast.  The arithmetic
// and its order are those of map_far32: groups of four lags from lo, each an
// explicit FMA chain, then single lags.
constexpr int kMapQ = 8;
// A wave's LDS: the staging of one-pixel tiles (two buffers of 64 lags: row
// fields, position) or the near band's queues.
template <int R>
__device__ __forceinline__ char* map_lds() {
  constexpr int kStage = R == 1 ? 2 * 64 * 3 * 16 : 0, kQueue = sizeof(NearQueue<kMapQ>);
  __shared__ __attribute__((aligned(16))) char lds[4][kStage > kQueue ? kStage : kQueue];
  return lds[threadIdx.x >> 6];
}

template <int M>
__device__ __forceinline__ void map_far32_r1(int lo, int hi, int64_t K, const float4* __restrict__ pos,
                                             const float* __restrict__ rows, float ex, float ey,
                                             float ee, double (&acc)[1]) {
  static_assert(M <= kMaxA, "row staging holds the 8 fields of degrees <= 3");
  if (lo >= hi) return;
  const int lane = threadIdx.x & 63;
  float4* const st = reinterpret_cast<float4*>(map_lds<1>());
  // lane i fetches lag base + i (clamped into [lo, hi))
  auto fetch = [&](int base, float4& r0, float4& r1, float4& pp) {
    const int n = min(base + lane, hi - 1);
    const float4* row = reinterpret_cast<const float4*>(rows + (int64_t)n * kRow32);
    r0 = row[0];
    r1 = row[1];
    pp = pos[K - n];
  };
  auto put = [&](int buf, const float4& r0, const float4& r1, const float4& pp) {
    float4* d = st + (buf * 64 + lane) * 3;
    d[0] = r0;
    d[1] = r1;
    d[2] = pp;
  };
  auto term = [&](int buf, int j, float& t) {
    const float4* d = st + (buf * 64 + j) * 3;
    const float4 u = d[0], v = d[1], p = d[2];
    const RowA row{u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
    const float a = __builtin_fmaf(ex, p.x, __builtin_fmaf(ey, p.y, ee + p.z));
    return series_f32a_q<M>(a, row, t);
  };
  float4 r0, r1, pp;
  fetch(lo, r0, r1, pp);
  put(0, r0, r1, pp);
  __builtin_amdgcn_wave_barrier();
  int buf = 0;
  for (int base = lo; base < hi; base += 64, buf ^= 1) {
    const int cnt = min(64, hi - base);
    const bool more = base + 64 < hi;
    if (more) fetch(base + 64, r0, r1, pp);
    int j = 0;
    for (; j + 4 <= cnt; j += 4) {
      float t0, t1, t2, t3;
      const float q0 = term(buf, j, t0), q1 = term(buf, j + 1, t1);
      const float q2 = term(buf, j + 2, t2), q3 = term(buf, j + 3, t3);
      float g = t0 * q0;
      g = __builtin_fmaf(t1, q1, g);
      g = __builtin_fmaf(t2, q2, g);
      g = __builtin_fmaf(t3, q3, g);
      acc[0] += (double)g;
    }
    for (; j < cnt; ++j) {
      float t;
      const float q = term(buf, j, t);
      acc[0] += (double)(t * q);
    }
    if (more) {
      __builtin_amdgcn_wave_barrier();
      put(buf ^ 1, r0, r1, pp);
      __builtin_amdgcn_wave_barrier();
    }
  }
}

template <int R, int U, bool MM>
__device__ __forceinline__ void map_far32_u(int M, int lo, int hi, int64_t K,
                                            const MapPos& pos,
                                            const float* __restrict__ rows,
                                            const MapPix<R, MM>& px,
                                            double (&acc)[R]) {
  switch (M) {
    case 0: map_far32<0, R, U, MM>(lo, hi, K, pos, rows, px, acc); break;
    case 1: map_far32<1, R, U, MM>(lo, hi, K, pos, rows, px, acc); break;
    case 2: map_far32<2, R, U, MM>(lo, hi, K, pos, rows, px, acc); break;
    case 3: map_far32<3, R, U, MM>(lo, hi, K, pos, rows, px, acc); break;
    case 4: map_far32<4, R, U, MM>(lo, hi, K, pos, rows, px, acc); break;
    case 5: map_far32<5, R, U, MM>(lo, hi, K, pos, rows, px, acc); break;
    default: map_far32<6, R, U, MM>(lo, hi, K, pos, rows, px, acc); break;
  }
}

template <int R, bool MM>
__device__ __forceinline__ void map_far32_seg(int M, int lo, int hi, int64_t K,
                                              const MapPos& pos, const float* __restrict__ rows,
                                              const MapPix<R, MM>& px, double (&acc)[R]) {
  // One pixel per lane: degrees <= 3 from rows staged in LDS; higher degrees
  // eight lags per step for more loads in flight.  The sum runs over groups
  // of four in lag order either way, so the result does not depend on the
  // tile width.
  if constexpr (R == 1) {
    float ex, ey;
    const float ee = px.ee[0];
    if constexpr (MM) {
      ex = (float)px.hi[0][0] + (float)px.lo[0][0];
      ey = (float)px.hi[0][1] + (float)px.lo[0][1];
    } else {
      ex = px.ex[0];
      ey = px.ey[0];
    }
    switch (M) {
      case 0: map_far32_r1<0>(lo, hi, K, pos.full, rows, ex, ey, ee, acc); return;
      case 1: map_far32_r1<1>(lo, hi, K, pos.full, rows, ex, ey, ee, acc); return;
      case 2: map_far32_r1<2>(lo, hi, K, pos.full, rows, ex, ey, ee, acc); return;
      case 3: map_far32_r1<3>(lo, hi, K, pos.full, rows, ex, ey, ee, acc); return;
      default: break;
    }
    const int mid = lo + ((hi - lo) & ~7);
    map_far32_u<R, 8, MM>(M, lo, mid, K, pos, rows, px, acc);
    lo = mid;
  }
  map_far32_u<R, 4, MM>(M, lo, hi, K, pos, rows, px, acc);
}

// Near band: per-pair choice.  A pixel tile lies together, so pairs of dx up to
// kMidDx come in whole waves and take the FP64 series in place, its row in
// scalar registers; the few beyond are queued as in do_arrival_near.  (512 maps
// of 128x128 over a 64x64 raster scan: 3.6 ms with the general form where it
// occurs, 4.4 with all of its pairs queued, whose evaluation gathers a row per
// lane, 3.3 now.)
template <int R, bool MM>
__device__ __forceinline__ void map_near32(int lo, int hi, int64_t K, const MapPos& pos,
                                           const double* __restrict__ rows64,
                                           const float* __restrict__ rows32,
                                           const MapPix<R, MM>& px, double (&acc)[R]) {
  const int lane = threadIdx.x & 63;
  NearQueue<kMapQ>& Q = *reinterpret_cast<NearQueue<kMapQ>*>(map_lds<R>());
  // lags as differences from lo: queue entries hold 29 bits
  rows64 += (int64_t)lo * kRow64;
  rows32 += (int64_t)lo * kRow32;
  int cnt = 0;
  // general-form terms have their own sum, so that a pixel's result does not
  // depend on when its queue is emptied (on the tile width)
  double gen[R];
#pragma unroll
  for (int r = 0; r < R; ++r) gen[r] = 0.0;
  wave_sync();
  MapVisits<MM> pn = map_visits<MM>(pos, K, lo);
  float cc[4], rhi[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const float* row = rows32 + (int64_t)min(s, hi - 1 - lo) * kRow32;
    cc[s] = ldc(row + kR32_C);
    rhi[s] = ldc(row + kR32_RHI);
  }
  for (int n = 0; n < hi - lo; n += 4) {
    const MapVisits<MM> p = pn;
    pn = map_visits<MM>(pos, K, lo + n + 4);
    f32x4_t a[R];
#pragma unroll
    for (int r = 0; r < R; ++r) a[r] = map_dist<R, true>(p, px, r);
    float c0[4], h0[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      c0[s] = cc[s];
      h0[s] = rhi[s];
      const float* row = rows32 + (int64_t)min(n + 4 + s, hi - 1 - lo) * kRow32;
      cc[s] = ldc(row + kR32_C);
      rhi[s] = ldc(row + kR32_RHI);
    }
    // not unrolled (one copy of the flush); the four lags move up in turn
#pragma unroll 1
    for (int s = 0; s < min(4, hi - lo - n); ++s) {
      if (__ballot(cnt > kMapQ - R)) near_flush<R>(Q, cnt, rows64, rows32, gen);
      const float* row = rows32 + (int64_t)(n + s) * kRow32;
      bool low[R], mid[R], any_low = false, any_mid = false;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const float d = a[r][0], z = d * c0[0];
        const bool in = d * h0[0] <= kCull32Log2;
        low[r] = z <= kThr32;
        mid[r] = !low[r] && in && z <= kMidDx;
        any_low = any_low || low[r];
        any_mid = any_mid || mid[r];
        if (in && z > kMidDx) {
          Q.a[cnt][lane] = d;
          Q.n[cnt][lane] = (n + s) | (r << 29);
          ++cnt;
        }
      }
      if (__ballot(any_low)) {
        float w[kRow32];
#pragma unroll
        for (int k = 0; k < kRow32; ++k) w[k] = ldc(row + k);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const float v = series_f32<kMNear32>(a[r][0], w);
          acc[r] += low[r] ? (double)v : 0.0;
        }
      }
      if (__ballot(any_mid)) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const double v = phi_mid_mixed(a[r][0], rows64 + (int64_t)(n + s) * kRow64, row);
          acc[r] += mid[r] ? v : 0.0;
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) a[r] = f32x4_t{a[r][1], a[r][2], a[r][3], 0.0f};
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        c0[q] = c0[q + 1];
        h0[q] = h0[q + 1];
      }
    }
  }
  if (__ballot(cnt > 0)) near_flush<R>(Q, cnt, rows64, rows32, gen);
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] += gen[r];
}

// NEAR: a near-band item or a far one; MM: distances from the matrix cores.
template <int R, bool NEAR, bool MM>
__device__ __forceinline__ void do_map(const MapItem& item, const MapTime& tm,
                                       const MapPos& pos,
                                       const double* __restrict__ rows64,
                                       const float* __restrict__ rows32, double X0, double Y0,
                                       double DX, double DY, int W, int H,
                                       double* __restrict__ partial) {
  const int lane = threadIdx.x & 63;
  const int64_t npix = (int64_t)W * H;
  const int64_t p0 = (int64_t)item.tile * (64 * R) + (int64_t)R * lane;
  double acc[R];
  MapPix<R, MM> px;
  bool wide = false;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t pix = min(p0 + r, npix - 1);
    const float x = (float)(X0 + (double)(pix % W) * DX);
    const float y = (float)(Y0 + (double)(pix / W) * DY);
    px.ee[r] = __builtin_fmaf(y, y, x * x);
    if constexpr (MM) {
      const _Float16 xh = (_Float16)x, yh = (_Float16)y;
      const _Float16 xl = (_Float16)(x - (float)xh), yl = (_Float16)(y - (float)yh);
      px.hi[r] = half4_t{xh, yh, (_Float16)4096.0f, (_Float16)1.0f};
      px.lo[r] = half4_t{xl, yl, (_Float16)0.0f, (_Float16)0.0f};
      wide = wide || xl != (_Float16)0.0f || yl != (_Float16)0.0f;
    } else {
      px.ex[r] = x;
      px.ey[r] = y;
    }
    acc[r] = 0.0;
  }
  if constexpr (MM) px.wide = __ballot(wide) != 0;
  const double* r64b = rows64 + tm.row_base * kRow64;
  const float* r32b = rows32 + tm.row_base * kRow32;
  if constexpr (NEAR) {
    if (item.n_lo < item.n_hi)
      map_near32<R, MM>(item.n_lo, item.n_hi, tm.K, pos, r64b, r32b, px, acc);
  } else {
    for (int M = tm.bounds.m_max; M >= 0; --M) {
      int lo, hi;
      seg_range(tm.bounds, M, item.n_lo, item.n_hi, lo, hi);
      if (lo < hi) map_far32_seg<R, MM>(M, lo, hi, tm.K, pos, r32b, px, acc);
    }
  }
  double* out = partial + (tm.slot_base + item.slot) * npix;
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (p0 + r < npix) out[p0 + r] = acc[r];
}

}  // namespace dd
