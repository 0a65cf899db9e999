// dd_gauss.h -- FP64 maps as sums of separable Gaussians: shared types of the
// host plan and the kernels of dd_gauss.hip.  Not part of the public ABI.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "dd_internal.h"

namespace dd {

// Pixels of a tile of a narrow map: two per lane.
constexpr int kGaussRow = 128;

// One map: the visits started before its time, its pixel grid, the split of
// the work into items and where results go.  The visits are those of a scan
// (pos: double2 by visit in pitch units, lag (K - i) + f dwells) or of a list
// (pos: double4 (x, y, t0, dwell) in start order, lag t - t0); the most
// recent one is visit i_last, and visits i_last, i_last - 1, ... (n of them)
// contribute.  With b = s2 + k4 lag, a pair's x1 is |r - r_i|^2 is2 / b.
struct GaussJob {
  const void* pos;
  int64_t i_last, n;
  double K, f, t;
  double s2, k4, is2;
  double X0, Y0, DX, DY;  // pixel (u, v) at (X0 + u DX, Y0 + v DY)
  int32_t W, H;
  int32_t tiles_x, tiles;  // tiles of 16 F x 16 F pixels, or (F = 0) of kGaussRow in a row
  int32_t base, near;      // chunks of visits (see GaussChunks)
  int32_t n_chunks, F;
  double* partial;         // [n_chunks][W * H]
  double* out;             // [W * H]
  double pref;
  OutFlag fl, fl2;         // the handle's flag and, in a batch, the call's
};

// Chunks of a map's visits, by recency r = 0 (the last started), 1, ...:
// with `near`, the 64 most recent visits in chunks of 2, 2, 4, 8, 16 and 32
// (they take up to a few dozen Gaussians each), then `base` visits each.
struct GaussChunks {
  __host__ __device__ static int32_t count(int64_t n, int32_t base, int32_t near) {
    if (n <= 0) return 1;  // one (empty) chunk: its partial sums are zeros
    if (!near) return (int32_t)((n + base - 1) / base);
    if (n <= 2) return 1;
    int32_t c = 1;
    for (int64_t e = 2; e < n && e < 64; e *= 2) ++c;
    if (n > 64) c += (int32_t)((n - 64 + base - 1) / base);
    return c;
  }
  __host__ __device__ static void range(int32_t c, int64_t n, int32_t base, int32_t near,
                                        int64_t& r0, int64_t& r1) {
    if (!near) {
      r0 = (int64_t)c * base;
      r1 = r0 + base;
    } else if (c < 6) {
      r0 = c == 0 ? 0 : (int64_t)1 << c;
      r1 = (int64_t)2 << c;
    } else {
      r0 = 64 + (int64_t)(c - 6) * base;
      r1 = r0 + base;
    }
    if (r1 > n) r1 = n;
  }
};

// Partial sums of the maps of one launch group in calls of many maps (256 MiB).
constexpr int64_t kGaussGroup = (int64_t)1 << 25;

// Split of maps of w x h pixels over at most n_vis visits, n_t of them in the
// call: tile side 16 F (0: kGaussRow pixels in a row) and visits per chunk.
struct GaussShape {
  int32_t F, base, near;
};
GaussShape gauss_shape(int64_t w, int64_t h, int64_t n_vis, int64_t n_t);

// The job of block (x, y) of a grid of n_jobs by the jobs' blocks; y is the block of
// the job.  The same blocks of all jobs are dealt out together, the recent (long)
// chunks first, to the 32 shader engines in turn; the rotation by y keeps an engine
// from having the same jobs, whose numbers of visits differ, in every row.  (A row
// per job gave an engine the same chunks of every job in grids of 16, 32, .. blocks a
// job: 384 maps of 1000x1 pixels of a 256x256 scan 60 ms, 16.6 so.)
// x < n_jobs; x + y fits 32 bits.  The division is left to calls of few jobs and many
// blocks (64 maps of 32x32: 23.5 us with a 64-bit one at the start of every block,
// 23.0 so).
__host__ __device__ inline uint32_t gauss_job_of(uint32_t x, uint32_t y, uint32_t n_jobs) {
  uint32_t j = x + y;
  if (j >= n_jobs) j -= n_jobs;
  return j < n_jobs ? j : j % n_jobs;
}

// Fills the tile and chunk fields of a job whose grid and n are set.
inline void gauss_split(GaussJob& j, const GaussShape& s) {
  const int32_t T = 16 * s.F;
  j.F = s.F;
  j.tiles_x = T ? (j.W + T - 1) / T : 0;
  j.tiles = T ? j.tiles_x * ((j.H + T - 1) / T) : (int32_t)(((int64_t)j.W * j.H + kGaussRow - 1) / kGaussRow);
  j.base = s.base;
  j.near = s.near;
  j.n_chunks = GaussChunks::count(j.n, s.base, s.near);
}

// Partial sums of n_jobs maps (device array, all with tile factor F) of
// scans (vis = false) or visit lists; `items` is the largest tiles * n_chunks
// among them.  Then their outputs: pref times the sum of a pixel's chunks.
hipError_t launch_gauss_map(const GaussJob* jobs, int32_t n_jobs, int64_t items, int32_t F,
                            bool vis, hipStream_t st);
hipError_t launch_gauss_reduce(const GaussJob* jobs, int32_t n_jobs, int64_t max_pixels,
                               hipStream_t st);

}  // namespace dd
