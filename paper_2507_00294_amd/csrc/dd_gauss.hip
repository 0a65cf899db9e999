// dd_gauss.hip -- FP64 maps on the matrix cores, as sums of separable
// Gaussians.
//
// A visit's field at squared distance a (Eqs. 1-2; b0, b1 its b at the end and
// the start of its beam-on time) is
//   E1(a/b1) - E1(a/b0) = int e^{-a beta} dbeta / beta over [1/b1, 1/b0]
//                       = int_0^L e^{-a e^s / b1} ds,  L = ln(b1/b0),
// which a Gauss-Legendre rule in s turns into a few Gaussians, omega_k
// e^{-beta_k a}.  On a pixel grid a Gaussian is a product of a factor of the
// column and one of the row, so a map is the matrix product
//   psi(v, u) = sum_{i,k} [omega_ik e^{-beta_ik (Y_v - y_i)^2}] [e^{-beta_ik (X_u - x_i)^2}]
// over all (visit, node) pairs: one FP64 multiply-add per pixel, visit and
// node instead of a series and an exponential.  All terms are positive and
// the rules are good to 5e-15 of each visit's own term at every distance (see
// gauss_nodes), so the sum keeps its relative accuracy at every pixel, also
// where all terms are tiny.
//
// A wave owns a tile of 16 F x 16 F pixels and a chunk of visits.  It takes 64
// visits at a time, one per lane, drops those that are beyond the cull for the
// whole tile, chooses the number of nodes by the tile's distances, and then,
// node by node, feeds four visits per v_mfma_f64_16x16x4: each lane evaluates
// the F column and F row factors of its visit (k = lane / 16) and pixel
// coordinate (lane % 16) in registers.
//
// Maps of one or two rows or columns leave most of a tile empty.  They go 128
// pixels at a time in row order (F = 0), two per lane and two nodes at a time, each
// Gaussian of the squared distance in one exponential and added by a vector
// multiply-add.
//
// Bound: the FP64 pipe.  A v_mfma_f64_16x16x4 takes about 72 cycles and an FP64
// vector operation 4, and the two do not overlap, not even from different
// waves (measured); a step is F^2 MFMAs and 2 F exponentials of 18 operations,
// i.e. 1150 + 630 cycles at F = 4 and 72 + 160 at F = 1, which is why F is as
// large as the call's work allows.  Measured against a per-pair series with
// its own exponential (25 to 60 FP64 operations a pair), random order: the final
// map of a 256x256 scan (4.3e9 pairs) 6.4 -> 0.84 ms, 512 maps of 128x128 over a
// 64x64 scan 28.8 -> 3.2 ms, 64 maps of 32x32 of an 8x8 scan 104 -> 53 us.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "dd_device.h"
#include "dd_gauss.h"
#include "dd_log.h"
#include "dd_visit_rows.h"

namespace dd {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// Gauss-Legendre rules of 2 .. 16 nodes on [0, 1]; rule N at N (N - 1) / 2 - 1.
constexpr int kMaxNodes = 16;
constexpr int kRuleLen = kMaxNodes * (kMaxNodes + 1) / 2 - 1;
struct GaussRules {
  double z[kRuleLen], w[kRuleLen];
  template <int N>
  constexpr void put() {
    constexpr GLRule<N> g{};
    for (int k = 0; k < N; ++k) {
      z[N * (N - 1) / 2 - 1 + k] = g.x[k];
      w[N * (N - 1) / 2 - 1 + k] = g.w[k];
    }
    if constexpr (N < kMaxNodes) put<N + 1>();
  }
  constexpr GaussRules() : z(), w() { put<2>(); }
};
__constant__ GaussRules kRules{};

// Coefficients of the degree-D polynomial for 2^h on |h| <= 1/2 that is left
// when the Taylor series' terms of degree D + 8 down to D + 1 are each replaced
// by the lower-degree part of h^n - T_n(2h) / 2^{2n-1} (economization).  What
// is dropped is (ln 2)^n / n! / 2^{2n-1} per degree: 2e-16 for D = 10, less than
// a rounding for D = 12.  Interpolating in double precision instead leaves the constant
// term 1.7e-15 off.
template <int D>
struct Exp2Econ {
  double c[D + 1];
  constexpr Exp2Econ() : c() {
    constexpr int N = D + 8;
    double t[N + 1] = {};
    t[0] = 1.0;
    for (int k = 1; k <= N; ++k) t[k] = t[k - 1] * kLn2 / k;
    for (int n = N; n > D; --n) {
      // T_n's coefficients (integers, exact) in x = 2h
      double a[N + 1] = {}, b[N + 1] = {};
      a[0] = 1.0;
      b[1] = 1.0;
      for (int k = 2; k <= n; ++k) {
        double e[N + 1] = {};
        for (int m = 0; m <= k; ++m) e[m] = (m > 0 ? 2.0 * b[m - 1] : 0.0) - a[m];
        for (int m = 0; m <= N; ++m) {
          a[m] = b[m];
          b[m] = e[m];
        }
      }
      // b[n] x^n = 2^{2n-1} h^n: subtract t[n] / 2^{2n-1} T_n(2h)
      double scale = t[n] / b[n];
      for (int m = 0; m < n; ++m) scale *= 0.5;
      double x = 1.0;  // 2^m
      for (int m = 0; m <= n; ++m, x *= 2.0) t[m] -= scale * b[m] * x;
    }
    for (int k = 0; k <= D; ++k) c[k] = t[k];
  }
};

// 2^x: D = 10 (relative error 2e-16 besides roundings) for the pixels'
// factors, D = 12 for the nodes, where a relative error grows by the exponent
// of the node's Gaussian, up to 745.
template <int D>
__device__ __forceinline__ double gauss_exp2(double x) {
  constexpr Exp2Econ<D> e{};
  const double m = __builtin_rint(x);
  const double h = x - m;
  double p = e.c[D];
#pragma unroll
  for (int k = D - 1; k >= 0; --k) p = fma(p, h, e.c[k]);
  return __builtin_ldexp(p, (int)m);
}

// ln(1 + q) for 0 <= q < 1e300: ln_pos with m - 1 = q kept exact where 1 + q is
// below sqrt(2).  (The library's log1p and exp, inlined, cost this kernel its
// second wave per SIMD.)
__device__ __forceinline__ double gauss_log1p(double q) {
  constexpr ArtanhSeries a{};
  const double x = 1.0 + q;
  int e = (int)((__double_as_longlong(x) >> 52) & 0x7ff) - 1023;
  double m = __builtin_ldexp(x, -e);
  if (m > 1.4142135623730951) {
    m *= 0.5;
    ++e;
  }
  const double s = (e == 0 ? q : m - 1.0) / (m + 1.0), z = s * s;
  double p = a.c[10];
#pragma unroll
  for (int k = 9; k >= 0; --k) p = fma(p, z, a.c[k]);
  return fma((double)e, kLn2, s * p);
}

// Nodes for which one Gauss-Legendre rule on [0, L] has a relative error below
// 2.6e-15 for every a with a (1/b0 - 1/b1) <= dx (against the integral in 40
// digits: 1e-15 to 2.4e-15 at the ends of these ranges and L small, 2.6e-15 with
// 16 nodes at dx = 22, where the roundings of the nodes bring it to 4.5e-15); 0 if
// more than 16 are needed or L > 0.3: panels (below).
__device__ __forceinline__ int gauss_nodes(double L, double dx) {
  if (L > 0.3 || dx > 22.0) return 0;
  int n = dx <= 1.8e-3 ? 2
          : dx <= 3.9e-2 ? 3
          : dx <= 0.2 ? 4
          : dx <= 0.55 ? 5
          : dx <= 1.2 ? 6
          : dx <= 2.1 ? 7
          : dx <= 3.2 ? 8
          : dx <= 4.6 ? 9
          : dx <= 6.3 ? 10
          : dx <= 10.5 ? 12
          : dx <= 15.5 ? 14
                       : 16;
  // the rule must also resolve e^s over [0, L]
  if (L > 1e-3) n = max(n, L <= 0.01 ? 3 : L <= 0.1 ? 4 : 6);
  return n;
}
// Panels, for the few most recent visits: 16 nodes on each of [s_p, s_{p+1}]
// with s_p where x1max (e^s - 1) = 20 (5/2)^{p-1}, at most 2 long.  A panel's
// own rule error grows with its share of the exponent, but the panels before
// it carry a factor e^{20} and more of the sum by then.
__device__ __forceinline__ double gauss_panel_end(double s, double x1max, double& D, double L) {
  const double e = gauss_log1p(fmin(D / x1max, 1e299));
  double r = fmin(L, s + 2.0);
  if (e <= r) {
    r = e;
    D *= 2.5;
  }
  return r;
}

struct GaussVisit {
  double x, y;      // position
  double rb, L;     // is2 / b1, and the range of s used
  double x1max;     // largest x1 of a pixel of the tile that counts
  int nodes;        // 0: panels
  bool on;
};

// Beyond x1 = 745 both E1 values of a pair are below the double range; a
// margin keeps the roundings of the tile's bounds on the safe side.
constexpr double kGaussCull = kCullX64 * (1.0 + 1e-9);
// Parts of the integral that are e^{-37} (8e-17) of the whole at the tile's
// nearest pixel are left out.
constexpr double kGaussTail = 37.0;

template <bool VIS>
__device__ __forceinline__ GaussVisit gauss_visit(const GaussJob& j, int64_t r, const double4 box) {
  GaussVisit v;
  const int64_t i = j.i_last - r;
  double lag, on;
  if (VIS) {
    const double4 p = static_cast<const double4*>(j.pos)[i];
    v.x = p.x;
    v.y = p.y;
    lag = j.t - p.z;
    on = fmin(lag, p.w);
  } else {
    const double2 p = static_cast<const double2*>(j.pos)[i];
    v.x = p.x;
    v.y = p.y;
    lag = (j.K - (double)i) + j.f;
    on = fmin(lag, 1.0);
  }
  const double b0 = fma(j.k4, lag - on, j.s2), db = j.k4 * on;
  double q = db / b0;
  v.rb = j.is2 / (b0 + db);
  const double gx = fmax(0.0, fmax(box.x - v.x, v.x - box.y));
  const double gy = fmax(0.0, fmax(box.z - v.y, v.y - box.w));
  const double fx = fmax(fabs(box.x - v.x), fabs(box.y - v.x));
  const double fy = fmax(fabs(box.z - v.y), fabs(box.w - v.y));
  const double x1min = fma(gx, gx, gy * gy) * v.rb;
  v.x1max = fmin(fma(fx, fx, fy * fy) * v.rb, kGaussCull);
  v.on = lag > 0.0 && x1min <= kGaussCull;
  if (x1min * q > kGaussTail) q = kGaussTail / x1min;
  v.L = gauss_log1p(q);
  v.nodes = gauss_nodes(v.L, v.x1max * q);
  return v;
}

__device__ __forceinline__ void gauss_lds_sync() {
  // a wave's LDS operations complete in order: a compiler barrier at
  // wavefront scope orders its writes before other lanes' reads
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int kGaussLds = 64 + 4;  // visits of a stage, padded to whole MFMA steps
struct GaussStage {
  double2 xy[kGaussLds];
  double2 bw[kGaussLds];  // (-beta log2(e), omega) of the current node
};

// One node of the stage's n visits (in LDS): n / 4 MFMA steps.
template <int F>
__device__ __forceinline__ void gauss_node(const GaussStage& S, int n, int lane,
                                           const double (&px)[F], const double (&py)[F],
                                           f64x4 (&acc)[F][F]) {
  const int g = lane >> 4;
  for (int s = 0; s < n; s += 4) {
    const double2 xy = S.xy[s + g], bw = S.bw[s + g];
    double X[F], Y[F];
#pragma unroll
    for (int a = 0; a < F; ++a) {
      const double dx = px[a] - xy.x, dy = py[a] - xy.y;
      X[a] = gauss_exp2<10>(fmax(-1100.0, bw.x * (dx * dx)));
      Y[a] = bw.y * gauss_exp2<10>(fmax(-1100.0, bw.x * (dy * dy)));
    }
#pragma unroll
    for (int a = 0; a < F; ++a)
#pragma unroll
      for (int b = 0; b < F; ++b)
        acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(Y[a], X[b], acc[a][b], 0, 0, 0);
  }
}

// One or two nodes (NN; their (-beta log2(e), omega) in bw and bw2) of the stage's n
// visits for a row of pixels, two per lane.  FLAT: the tile lies in one row or column
// of the map, px is the coordinate along it, and xy holds a visit's coordinate along
// it and the square of its distance from it.  No clamp: coordinates are bounded,
// and below 2^-1075 the result is 0.
template <int NN, bool FLAT>
__device__ __forceinline__ void gauss_node_row(const GaussStage& S, const double2* bw2, int n,
                                               const double (&px)[2], const double (&py)[2],
                                               double (&acc)[2]) {
  for (int s = 0; s < n; s += 2) {  // (the stage is padded)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const double2 xy = S.xy[s + k], b = S.bw[s + k];
      double2 c{};
      if (NN == 2) c = bw2[s + k];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const double dx = px[q] - xy.x, dy = FLAT ? 0.0 : py[q] - xy.y;
        const double a = fma(dx, dx, FLAT ? xy.y : dy * dy);
        acc[q] = fma(b.y, gauss_exp2<10>(b.x * a), acc[q]);
        if (NN == 2) acc[q] = fma(c.y, gauss_exp2<10>(c.x * a), acc[q]);
      }
    }
  }
}

// Wave w of block (x, y): item 4 (block0 + y) + w of job gauss_job_of(x, y) -- tile
// item % tiles, chunk item / tiles (the recent visits, which take most nodes, first).
template <int F, bool VIS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(F == 4 ? 2 : F == 2 ? 3 : 4, 8)))
k_gauss_map(const GaussJob* __restrict__ jobs, uint32_t block0) {
  __shared__ GaussStage stages[4];
  __shared__ double2 seconds[F ? 1 : 4][F ? 1 : kGaussLds];  // F = 0: the second node of two
  const GaussJob& j = jobs[gauss_job_of(blockIdx.x, blockIdx.y, gridDim.x)];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t item = (int64_t)(block0 + blockIdx.y) * 4 + wave;
  if (item >= (int64_t)j.tiles * j.n_chunks) return;
  GaussStage& S = stages[wave];
  const int tile = (int)(item % j.tiles), chunk = (int)(item / j.tiles);
  int64_t r0, r1;
  GaussChunks::range(chunk, j.n, j.base, j.near, r0, r1);
  constexpr int N = F ? F : 2;
  int u0, u1, v0, v1;  // first and last column and row
  double px[N], py[N];
  const int64_t npix = (int64_t)j.W * j.H, p0 = (int64_t)tile * kGaussRow;
  if constexpr (F == 0) {
    const int64_t p1 = min(p0 + kGaussRow, npix) - 1;
    v0 = (int)(p0 / j.W);
    v1 = (int)(p1 / j.W);
    u0 = v0 == v1 ? (int)(p0 % j.W) : 0;
    u1 = v0 == v1 ? (int)(p1 % j.W) : j.W - 1;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int64_t p = min(p0 + lane + 64 * q, p1);
      px[q] = fmin(fmax(j.X0 + (double)(p % j.W) * j.DX, -1e130), 1e130);
      py[q] = fmin(fmax(j.Y0 + (double)(p / j.W) * j.DY, -1e130), 1e130);
    }
  } else {
    u0 = tile % j.tiles_x * (16 * F);
    v0 = tile / j.tiles_x * (16 * F);
    u1 = min(u0 + 16 * F, j.W) - 1;
    v1 = min(v0 + 16 * F, j.H) - 1;
#pragma unroll
    for (int a = 0; a < F; ++a) {
      px[a] = j.X0 + (double)min(u0 + 16 * a + (lane & 15), u1) * j.DX;
      py[a] = j.Y0 + (double)min(v0 + 16 * a + (lane & 15), v1) * j.DY;
    }
  }
  const double xa = j.X0 + (double)u0 * j.DX, xb = j.X0 + (double)u1 * j.DX;
  const double ya = j.Y0 + (double)v0 * j.DY, yb = j.Y0 + (double)v1 * j.DY;
  const double4 box = make_double4(fmin(xa, xb), fmax(xa, xb), fmin(ya, yb), fmax(ya, yb));
  f64x4 acc[N][N];
  double row_acc[2] = {0.0, 0.0};
  const bool flat = F == 0 && (v0 == v1 || u0 == u1);
  const double along[2] = {v0 == v1 ? px[0] : py[0], v0 == v1 ? px[N > 1] : py[N > 1]};
#pragma unroll
  for (int a = 0; a < F; ++a)
#pragma unroll
    for (int b = 0; b < F; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};

  for (int64_t r = r0, re; r < r1; r = re) {
    // the stages of the 64 most recent visits double from 2 on: a stage takes
    // as many nodes as its most recent visit needs
    re = r >= 64 ? r + 64 : r < 2 ? 2 : 2ll << (31 - __builtin_clz((int)r));
    re = min(re, r1);
    GaussVisit v{};
    if (r + lane < re) v = gauss_visit<VIS>(j, r + lane, box);
    const uint64_t live = __ballot(v.on);
    if (!live) continue;
    const int n = __popcll(live);
    const int slot = __popcll(live & ((1ull << lane) - 1));
    gauss_lds_sync();  // the previous stage is no longer read
    if (v.on) {
      double2 xy = make_double2(v.x, v.y);
      if (F == 0 && flat) {
        const double off = v0 == v1 ? py[0] - v.y : px[0] - v.x;
        xy = make_double2(v0 == v1 ? v.x : v.y, off * off);
      }
      S.xy[slot] = xy;
    }
    if (lane < 4) {  // the last step's idle entries
      S.xy[n + lane] = make_double2(0.0, 0.0);
      S.bw[n + lane] = make_double2(0.0, 0.0);
      if constexpr (F == 0) seconds[wave][n + lane] = make_double2(0.0, 0.0);
    }
    // the rule of the stage: what its visits need at most
    const bool panels = __ballot(v.on && v.nodes == 0) != 0;
    int nodes = kMaxNodes;
    if (!panels)
      while (nodes > 2 && !__ballot(v.on && v.nodes >= nodes)) --nodes;
    const int at = nodes * (nodes - 1) / 2 - 1;
    const double rl2 = -kLog2e * v.rb;
    double s0 = 0.0, D = 20.0;
    do {  // one rule on [0, L], or panel by panel until every lane's end at its L
      double s1 = v.L;
      if (panels) s1 = s0 < v.L ? gauss_panel_end(s0, v.x1max, D, v.L) : s0;
      auto put = [&](double2* to, int k) {
        const double s = fma(s1 - s0, kRules.z[at + k], s0);
        if (v.on)
          to[slot] = make_double2(rl2 * gauss_exp2<12>(kLog2e * s), (s1 - s0) * kRules.w[at + k]);
      };
      if constexpr (F == 0) {
        double2* const bw2 = seconds[wave];
        for (int k = 0; k < nodes; k += 2) {
          gauss_lds_sync();
          put(S.bw, k);
          if (k + 1 < nodes) put(bw2, k + 1);
          gauss_lds_sync();
          const bool two = k + 1 < nodes;
          if (flat)
            two ? gauss_node_row<2, true>(S, bw2, n, along, py, row_acc)
                : gauss_node_row<1, true>(S, bw2, n, along, py, row_acc);
          else
            two ? gauss_node_row<2, false>(S, bw2, n, px, py, row_acc)
                : gauss_node_row<1, false>(S, bw2, n, px, py, row_acc);
        }
      } else {
        for (int k = 0; k < nodes; ++k) {
          gauss_lds_sync();
          put(S.bw, k);
          gauss_lds_sync();
          gauss_node<F>(S, n, lane, px, py, acc);
        }
      }
      s0 = s1;
    } while (panels && __ballot(v.on && s0 < v.L));
  }
  double* out = j.partial + (int64_t)chunk * npix;
  if constexpr (F == 0) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (p0 + lane + 64 * q < npix) out[p0 + lane + 64 * q] = row_acc[q];
    return;
  }
  // D element v of a lane: row 4 v + lane / 16, column lane % 16
#pragma unroll
  for (int a = 0; a < F; ++a)
#pragma unroll
    for (int b = 0; b < F; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = v0 + 16 * a + 4 * e + (lane >> 4), col = u0 + 16 * b + (lane & 15);
        if (row <= v1 && col <= u1) out[(int64_t)row * j.W + col] = acc[a][b][e];
      }
}

// 64 pixels per block, four threads each: thread g of a pixel adds chunks g,
// g + 4, ..., then the four sums in a fixed order.
__global__ void __launch_bounds__(256) k_gauss_reduce(const GaussJob* __restrict__ jobs) {
  __shared__ double part[4][64];
  const GaussJob& j = jobs[blockIdx.y];
  const int64_t npix = (int64_t)j.W * j.H;
  const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
  for (int64_t p0 = (int64_t)blockIdx.x * 64; p0 < npix; p0 += (int64_t)gridDim.x * 64) {
    const int64_t p = p0 + lane;
    double s = 0.0;
    if (p < npix)
      for (int c = g; c < j.n_chunks; c += 4) s += j.partial[(int64_t)c * npix + p];
    part[g][lane] = s;
    __syncthreads();
    if (g == 0 && p < npix) {
      const double v = j.pref * ((part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]));
      j.out[p] = v;
      flag_nonfinite(j.fl, v, p);
      flag_nonfinite(j.fl2, v, p);
    }
    __syncthreads();
  }
}

}  // namespace

// Larger tiles take fewer exponentials per multiply-add, smaller ones more
// waves: the largest tile that still gives the call about two waves per SIMD
// (2048 items), with chunks of at least 64 visits and at most ~130 per map --
// or a smaller one that leaves so much less of itself empty that a node of four
// visits takes fewer cycles for the whole map: 1780, 600 and 230 per tile for F =
// 4, 2, 1, and 600 per row of 128 pixels, where a call has 2048 items of them, or
// 1024 and they take half the cycles (one map of a 256x256 scan: 64x1 pixels, 128
// items, 373 us in rows, 157 with F = 1; 500x2, 1024 items, 393 and 240; 1x2048 of
// 4096 visits, 1024 items, 12 and 28 a map).  64 maps of a 64x64 scan, 4096x1 pixels:
// 5.9 ms with F = 4, 3.6 with F = 1, 1.0 in rows; 512x8: 0.89 with F = 4, 0.58 with
// F = 1; 8x8: 162 and 65 us.
// Where a call has more than 16k items of that kind (64k rows), chunks grow to
// leave about half as many.
// The 64 most recent visits of a map take up to a hundred nodes each, a million
// cycles of one wave at F = 4, as much as thousands of older ones: they have chunks of
// their own, unless the call's tiles alone are enough for every wave to have such a
// share.  Of a 64x64 scan, together and apart: 64 maps of 8x8 141 and 64 us, 256 of
// 33x33 660 and 485, 512 of 64x64 1170 and 1040; 4000 of 64x64 of an 8x8 scan 850
// and 920.  Partial sums: at most 32 kB an item, 1 GiB in all, or one chunk's for a
// call of more than 8k tiles.
GaussShape gauss_shape(int64_t w, int64_t h, int64_t n_vis, int64_t n_t) {
  auto up64 = [](int64_t v) { return (v + 63) / 64 * 64; };
  const int64_t base0 = std::max<int64_t>(64, up64((n_vis + 127) / 128));
  auto tiles = [&](int64_t F) {
    return F ? ((w + 16 * F - 1) / (16 * F)) * ((h + 16 * F - 1) / (16 * F)) : (w * h + kGaussRow - 1) / kGaussRow;
  };
  const int64_t chunks = (n_vis + base0 - 1) / base0;
  GaussShape s{1, (int32_t)base0, 1};
  for (int F : {4, 2})
    if (n_t * tiles(F) * chunks >= 2048) {
      s.F = F;
      break;
    }
  auto cycles = [&](int F) { return tiles(F) * (F == 4 ? 1780 : F == 2 ? 600 : F == 1 ? 230 : 600); };
  int64_t least = cycles(s.F);
  const int64_t row_items = n_t * tiles(0) * chunks;
  for (int F : {2, 1, 0})
    if (F < s.F && (F > 0 || row_items >= 2048 ? cycles(F) < least
                                               : row_items >= 1024 && 2 * cycles(F) < least)) {
      s.F = F;
      least = cycles(F);
    }
  const int64_t maps = n_t * tiles(s.F), most = s.F ? 16384 : 65536;
  if (maps >= (chunks > 1 ? 4096 : 2048)) s.near = 0;
  if (maps * chunks > most)
    s.base = (int32_t)std::min<int64_t>(
        up64(n_vis), std::max<int64_t>(base0, up64(n_vis / std::max<int64_t>(1, most / 2 / maps))));
  return s;
}

hipError_t launch_gauss_map(const GaussJob* jobs, int32_t n_jobs, int64_t items, int32_t F,
                            bool vis, hipStream_t st) {
  if (n_jobs <= 0 || items <= 0) return hipSuccess;
  if (F != 0 && F != 1 && F != 2 && F != 4) return hipErrorInvalidValue;
  const int64_t blocks = (items + 3) / 4;
  constexpr int32_t kJobs = 1 << 20, kBlocks = 32768;  // per launch
  for (int32_t k = 0; k < n_jobs; k += kJobs)
    for (int64_t b = 0; b < blocks; b += kBlocks) {
      const dim3 grid((unsigned)std::min(kJobs, n_jobs - k),
                      (unsigned)std::min<int64_t>(kBlocks, blocks - b));
      auto map = vis ? (F == 0   ? k_gauss_map<0, true>
                        : F == 1 ? k_gauss_map<1, true>
                        : F == 2 ? k_gauss_map<2, true>
                                 : k_gauss_map<4, true>)
                     : (F == 0   ? k_gauss_map<0, false>
                        : F == 1 ? k_gauss_map<1, false>
                        : F == 2 ? k_gauss_map<2, false>
                                 : k_gauss_map<4, false>);
      hipLaunchKernelGGL(map, grid, dim3(256), 0, st, jobs + k, (uint32_t)b);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

hipError_t launch_gauss_reduce(const GaussJob* jobs, int32_t n_jobs, int64_t max_pixels,
                               hipStream_t st) {
  if (n_jobs <= 0 || max_pixels <= 0) return hipSuccess;
  const unsigned bx = (unsigned)std::min<int64_t>((max_pixels + 63) / 64, 1 << 20);
  for (int32_t k = 0; k < n_jobs; k += 32768) {
    hipLaunchKernelGGL(k_gauss_reduce, dim3(bx, (unsigned)std::min(32768, n_jobs - k)), dim3(256),
                       0, st, jobs + k);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace dd
