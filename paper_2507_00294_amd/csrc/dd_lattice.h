// dd_lattice.h -- FP64 arrival queries of scans made of rasters: shared types of
// the host plan and the kernels of dd_lattice.hip.  Not part of the public ABI.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "dd_internal.h"

namespace dd {

// A scan as a sequence of rasters ("passes") of equal width: one (raster
// order), the frames (multi-frame) or the sub-lattices (interleaved, nx a
// multiple of the stride).  Visit first + r w + c of a pass is at (x0 + step c,
// y0 + step r).
//
// A class is an ordered pair of passes, the evaluated one and an earlier one
// (or itself): every pair of visits in it has lag dB + w dr + dc and
// displacement (ox + step dc, oy + step dr), dr and dc the differences of row
// and column, so its terms are a table over (dr, dc).  Frames are alike, so
// for them a class is a difference of frames.
struct LatClass {
  int64_t dB;
  int32_t ox, oy;
  int32_t hq;        // rows of the earlier pass
  int32_t same;      // the pass with itself: causal pairs only
  int32_t key0;      // its first row of the table; rows are dr = -(hq - 1) ..
                     // hp - 1, or 0 .. hp - 1 when `same`
};
// A pass: its sums take n_cls classes.  Frames add one class each to the
// frame before (n_frames > 1).  A block of k_lat_sum takes 64 columns of 16
// rows, or of 4 rows and its waves a quarter of the classes each, from
// kLatSplit classes on.
constexpr int kLatSplit = 4;
struct LatPass {
  int64_t first;
  int32_t cls, n_cls, h;
  int32_t block0;      // first block of k_lat_sum
};
struct LatJob {
  const LatClass* cls;
  const LatPass* passes;
  int32_t n_cls, n_passes, n_keys, n_blocks;
  int32_t w, step, n_frames;
  int64_t n_sum;         // visits per frame
  int32_t kf;            // lags below take the general form, the others the
  DegreeBounds bounds;   // series of their row's degree (as in the pair sums)
  const double* rows64;  // integer-lag rows
  double* sums;          // [n_keys][w]: a row of the table summed over columns
  double* out;
  double pref;
  OutFlag fl, fl2;       // the handle's flag and, in a batch, the call's
};

// The host's plan: the tables and the job's sizes (pointers, sums, out, flags:
// the caller's).
struct LatPlan {
  std::vector<LatClass> cls;
  std::vector<LatPass> passes;
  LatJob job{};
};

// One job, or n of them from a device array (max_keys, max_blocks and
// max_frame: the largest n_keys and n_blocks, and the largest n_sum of those
// with several frames, 0 if none has).
hipError_t launch_lattice(const LatJob& job, hipStream_t st);
hipError_t launch_lattice_batch(const LatJob* jobs, int32_t n, int32_t max_keys,
                                int32_t max_blocks, int64_t max_frame, hipStream_t st);

}  // namespace dd
