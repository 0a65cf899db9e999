// dd_lattice.hip -- FP64 arrival queries of raster, multi-frame and interleaved
// scans.
//
// Within a raster, and between two rasters of the same width, the displacement
// and the lag of a pair of visits depend on their difference of rows and
// columns (dr, dc) alone, so the pairs of Eq. 6 take only a table of distinct
// terms, about 2 w (2 h) per pair of rasters instead of (w h)^2 / 2:
//   psi(r, c) = sum over r', c' of g(r - r', c - c').
// k_lat_terms evaluates the table row by row (a block per dr) and sums each row
// over the columns a visit at column c sees, dc = c - w + 1 .. c: the sum of g
// up to dc = 0 from c - w + 1 (a suffix sum) plus the sum from 1 to c (a prefix
// sum).  k_lat_sum adds the rows a visit at row r sees, dr = r - h' + 1 .. r, the
// same way, and k_lat_frames the frames.  Every sum is of positive terms, none
// is a difference of prefix sums, so results keep their relative accuracy.
//
// Bound: launches and memory latency (a 512x512 raster has 5.2e5 terms for
// 3.4e10 pairs).  Against evaluating every pair: 8x8 raster 0.042 -> 0.018 ms,
// 64x64 0.33 -> 0.019, 512x512 24 -> 0.062, four frames of 97x101 0.86 -> 0.031,
// 32x32 interleaved at stride 2 0.31 -> 0.023.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "dd_device.h"
#include "dd_lattice.h"

namespace dd {

namespace {

constexpr int kLatMaxW = 2048;  // probes per side of a scan

// Sums v over the block's threads 0 .. t - 1 (exclusive), in a fixed order.
__device__ __forceinline__ double block_before(double v, double* buf) {
  const int t = threadIdx.x;
  buf[t] = v;
  __syncthreads();
  for (int d = 1; d < 256; d <<= 1) {
    const double u = t >= d ? buf[t - d] : 0.0;
    __syncthreads();
    buf[t] += u;
    __syncthreads();
  }
  const double r = t > 0 ? buf[t - 1] : 0.0;
  __syncthreads();
  return r;
}

// The term of squared distance a and lag n as the pair sums evaluate it, so
// that a visit range of the same scan adds up the same terms.
__device__ __forceinline__ double lat_term(const LatJob& j, double a, int64_t n) {
  const double* row = j.rows64 + n * kRow64;
  if (n < j.kf) return phi_general_f64(a, row);
  int M = 0;
  while (M < j.bounds.m_max && n < j.bounds.b[M]) ++M;
  const double z = a * row[kR64_C];
  double q = row[kR64_P + M];
  for (int m = M - 1; m >= 0; --m) q = fma(q, z, row[kR64_P + m]);
  return exp2_neg9(a * row[kR64_RL2]) * q;
}

__device__ __forceinline__ void lat_terms(const LatJob& j, int key) {
  __shared__ double g[2 * kLatMaxW];
  __shared__ double buf[256];
  int lo = 0;
  for (int hi = j.n_cls - 1; lo < hi;) {  // the key's class
    const int mid = (lo + hi + 1) >> 1;
    if (j.cls[mid].key0 <= key)
      lo = mid;
    else
      hi = mid - 1;
  }
  const LatClass k = j.cls[lo];
  const int w = j.w, dr = key - k.key0 - (k.same ? 0 : k.hq - 1);
  const int64_t n0 = k.dB + (int64_t)w * dr;
  const double dy = (double)(k.oy + j.step * dr);
  const int t = threadIdx.x;
  for (int i = t; i < 2 * w - 1; i += 256) {
    const int dc = i - (w - 1);
    double v = 0.0;
    if (!(k.same && dr == 0 && dc <= 0)) {
      const double dx = (double)(k.ox + j.step * dc);
      v = lat_term(j, fma(dx, dx, dy * dy), n0 + dc);
    }
    g[i] = v;
  }
  __syncthreads();
  // thread t owns columns [t len, (t + 1) len): suffix sums over i = 0 .. w - 1
  // (dc <= 0) and prefix sums over i = w .. 2 w - 2 (dc = 1 .. w - 1)
  const int len = (w + 255) / 256;
  const int c0 = min(t * len, w), c1 = min(c0 + len, w);
  // suffix: thread 255 - t's share in reversed order, so that "before" is "after"
  const int s1 = w - c0, s0 = w - c1;  // columns [s0, s1)
  double sum = 0.0;
  for (int c = s1 - 1; c >= s0; --c) sum += g[c];
  double run = block_before(sum, buf);
  for (int c = s1 - 1; c >= s0; --c) {
    run += g[c];
    g[c] = run;  // only this thread reads g[s0 .. s1)
  }
  sum = 0.0;
  for (int c = max(c0, 1); c < c1; ++c) sum += g[w - 1 + c];
  run = block_before(sum, buf);  // also: every suffix sum is written
  double* out = j.sums + (int64_t)key * w;
  for (int c = c0; c < c1; ++c) {
    if (c > 0) run += g[w - 1 + c];
    out[c] = g[c] + run;
  }
}

// The classes q, q + step, .. of a pass, summed for rows r0 .. r0 + 3 of column c.
__device__ __forceinline__ void lat_classes(const LatJob& j, const LatPass& P, int q, int step,
                                            int r0, int c, double (&acc)[4]) {
  const int nr = min(4, P.h - r0);
  for (q += P.cls; q < P.cls + P.n_cls; q += step) {
    const LatClass k = j.cls[q];
    // row dr of the class at this column
    const double* h = j.sums + ((int64_t)k.key0 + (k.same ? 0 : k.hq - 1)) * j.w + c;
    auto at = [&](int dr) { return h[(int64_t)dr * j.w]; };
    // rows dr = 1 (0 when `same`) .. r0, then one more per row
    double up = 0.0;
#pragma unroll 8
    for (int dr = k.same ? 0 : 1; dr <= r0; ++dr) up += at(dr);
    // rows dr = r - hq + 1 .. 0: from the last row of the four upwards
    double down[4] = {0.0, 0.0, 0.0, 0.0};
    if (!k.same) {
      double d = 0.0;
#pragma unroll 8
      for (int dr = 0; dr > r0 + 3 - k.hq + 1; --dr) d += at(dr);
#pragma unroll
      for (int i = 3; i >= 0; --i) {
        const int dr = r0 + i - k.hq + 1;
        if (dr <= 0) d += at(dr);
        down[i] = d;
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i > 0 && i < nr) up += at(r0 + i);
      acc[i] += down[i] + up;
    }
  }
}

__device__ __forceinline__ void lat_put(const LatJob& j, int64_t o, double v) {
  v *= j.pref;
  j.out[o] = v;
  flag_nonfinite(j.fl, v, o);
  flag_nonfinite(j.fl2, v, o);
}

__device__ __forceinline__ void lat_sum(const LatJob& j, int block) {
  __shared__ double part[3][4][64];
  int lo = 0;
  for (int hi = j.n_passes - 1; lo < hi;) {  // the block's pass
    const int mid = (lo + hi + 1) >> 1;
    if (j.passes[mid].block0 <= block)
      lo = mid;
    else
      hi = mid - 1;
  }
  const LatPass P = j.passes[lo];
  const int ctiles = (j.w + 63) / 64, b = block - P.block0;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = b % ctiles * 64 + lane;
  const bool split = P.n_cls >= kLatSplit;
  const int r0 = split ? b / ctiles * 4 : b / ctiles * 16 + 4 * wave;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if (r0 < P.h) lat_classes(j, P, split ? wave : 0, split ? 4 : 1, r0, min(c, j.w - 1), acc);
  if (split) {
    if (wave > 0)
#pragma unroll
      for (int i = 0; i < 4; ++i) part[wave - 1][i][lane] = acc[i];
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] += part[0][i][lane] + part[1][i][lane] + part[2][i][lane];
  }
  if (c >= j.w) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (r0 + i >= P.h) break;
    const int64_t o = P.first + (int64_t)(r0 + i) * j.w + c;
    if (j.n_frames > 1)
      j.out[o] = acc[i];
    else
      lat_put(j, o, acc[i]);
  }
}

// Frames: each adds its class to the frame before.
__device__ __forceinline__ void lat_frames(const LatJob& j, int64_t i) {
  if (i >= j.n_sum) return;
  double sum = 0.0;
  for (int f = 0; f < j.n_frames; f += 8) {
    const int m = min(8, j.n_frames - f);
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = j.out[(int64_t)(f + min(k, m - 1)) * j.n_sum + i];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (k >= m) break;
      sum += v[k];
      lat_put(j, (int64_t)(f + k) * j.n_sum + i, sum);
    }
  }
}

__global__ void __launch_bounds__(256) k_lat_terms(LatJob j) { lat_terms(j, blockIdx.x); }
__global__ void __launch_bounds__(256) k_lat_sum(LatJob j) { lat_sum(j, blockIdx.x); }
__global__ void __launch_bounds__(64) k_lat_frames(LatJob j) {
  lat_frames(j, (int64_t)blockIdx.x * 64 + threadIdx.x);
}
__global__ void __launch_bounds__(256) k_lat_terms_batch(const LatJob* __restrict__ jobs) {
  const LatJob& j = jobs[blockIdx.y];
  if ((int)blockIdx.x < j.n_keys) lat_terms(j, blockIdx.x);
}
__global__ void __launch_bounds__(256) k_lat_sum_batch(const LatJob* __restrict__ jobs) {
  const LatJob& j = jobs[blockIdx.y];
  if ((int)blockIdx.x < j.n_blocks) lat_sum(j, blockIdx.x);
}
__global__ void __launch_bounds__(64) k_lat_frames_batch(const LatJob* __restrict__ jobs) {
  const LatJob& j = jobs[blockIdx.y];
  if (j.n_frames > 1) lat_frames(j, (int64_t)blockIdx.x * 64 + threadIdx.x);
}

}  // namespace

hipError_t launch_lattice(const LatJob& job, hipStream_t st) {
  if (job.w < 1 || job.w > kLatMaxW || job.n_keys < 1 || job.n_blocks < 1)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_lat_terms, dim3(job.n_keys), dim3(256), 0, st, job);
  hipLaunchKernelGGL(k_lat_sum, dim3(job.n_blocks), dim3(256), 0, st, job);
  if (job.n_frames > 1)
    hipLaunchKernelGGL(k_lat_frames, dim3((unsigned)((job.n_sum + 63) / 64)), dim3(64), 0, st, job);
  return hipGetLastError();
}

hipError_t launch_lattice_batch(const LatJob* jobs, int32_t n, int32_t max_keys,
                                int32_t max_blocks, int64_t max_frame, hipStream_t st) {
  for (int32_t k = 0; k < n; k += 32768) {
    const unsigned m = (unsigned)(n - k < 32768 ? n - k : 32768);
    hipLaunchKernelGGL(k_lat_terms_batch, dim3(max_keys, m), dim3(256), 0, st, jobs + k);
    hipLaunchKernelGGL(k_lat_sum_batch, dim3(max_blocks, m), dim3(256), 0, st, jobs + k);
    if (max_frame > 0)
      hipLaunchKernelGGL(k_lat_frames_batch, dim3((unsigned)((max_frame + 63) / 64), m), dim3(64), 0,
                         st, jobs + k);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace dd
