// unet_kernels.hip -- elementwise kernels of the learned surrogate (the
// convolutions: unet_conv.hip; their gradients: unet_wgrad.hip): the
// relative-L2 loss, gradient-norm clipping, Adam with FP32 master weights and
// the rearrangement of the weights into the convolution's BF16 layouts, the
// dihedral mini-batch gather of training, and the surrogate's input gather,
// output transform and spot-check.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "unet_kernels.h"

namespace dd {
namespace nn {

// Loss of a batch of maps (one block per map of n pixels).  The prediction
// is own + exp(y) (exp argument capped at 80); map b's loss is its squared
// relative L2 error |pred - t|^2 / |t|^2, written to loss_map[b].  The
// objective whose gradient dy is returned (for the mean over maps) adds the
// anchor (anchor / n) sum_i (r_i / t_i)^2 (y_i - ln r_i)^2 with r_i = max(t_i
// - own_i, 1e-6 t_i): the same per-pixel weight as the relative error, but a
// gradient that does not vanish when exp(y) is far below r.  Sums are in
// double, in a fixed order.
__global__ void __launch_bounds__(256) k_rel_l2(const float* __restrict__ y,
                                                const float* __restrict__ own,
                                                const float* __restrict__ t, int n, float inv_maps,
                                                float anchor, float* __restrict__ dy,
                                                double* __restrict__ loss_map) {
  __shared__ double red[256];
  const int64_t base = (int64_t)blockIdx.x * n;
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) {
    const double ti = t[base + i];
    s += ti * ti;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  const double den = red[0] > 0.0 ? red[0] : 1.0;
  __syncthreads();
  const float scale = (float)(2.0 / den) * inv_maps;
  const float ascale = 2.0f * anchor / (float)n * inv_maps;
  double num = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) {
    const float yi = y[base + i], ti = t[base + i], oi = own[base + i];
    const float e = __expf(fminf(yi, 80.0f));
    const float d = oi + e - ti;
    num += (double)d * d;
    float g = scale * d * e;
    if (ti > 0.f) {
      const float r = fmaxf(ti - oi, 1e-6f * ti), wr = r / ti;
      g += ascale * wr * wr * (yi - __logf(r));
    }
    dy[base + i] = g;
  }
  red[threadIdx.x] = num;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss_map[blockIdx.x] = red[0] / den;
}

// Sum of squares of g: one partial per block (the grid has kNormBlocks blocks).
__global__ void __launch_bounds__(256) k_sumsq(const float* __restrict__ g, int64_t n,
                                               double* __restrict__ partial) {
  __shared__ double red[256];
  double s = 0.0;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x)
    s += (double)g[e] * g[e];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// scale_norm[0] = min(1, clip / |g|) (1 when clip <= 0, 0 when |g| is not
// finite, which skips the update); scale_norm[1] = |g|.
__global__ void __launch_bounds__(256) k_clip_scale(const double* __restrict__ partial, float clip,
                                                    float* __restrict__ scale_norm) {
  __shared__ double red[256];
  red[threadIdx.x] = partial[threadIdx.x];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double norm = sqrt(red[0]);
    double sc = 1.0;
    if (clip > 0.f && norm > clip) sc = clip / norm;
    if (!(norm <= 1e300)) sc = 0.0;
    scale_norm[0] = (float)sc;
    scale_norm[1] = (float)norm;
  }
}

// Adam with FP32 master weights (bias-corrected) on the scaled gradient
// g * scale[0].  bc1 = 1 - beta1^t, bc2 = 1 - beta2^t.
__global__ void __launch_bounds__(256) k_adam(float* __restrict__ w, float* __restrict__ m,
                                              float* __restrict__ v, const float* __restrict__ g,
                                              const float* __restrict__ scale, int64_t n, float lr,
                                              float b1, float b2, float eps, float bc1, float bc2) {
  const float sc = scale[0];
  if (sc == 0.f) return;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[e] * sc;
    const float mi = b1 * m[e] + (1.0f - b1) * gi;
    const float vi = b2 * v[e] + (1.0f - b2) * gi * gi;
    m[e] = mi;
    v[e] = vi;
    w[e] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
  }
}

// BF16 weight layouts of the convolutions from the FP32 master vector (layer
// blockIdx.y), whose weights W[k][j] (k = tap ci + c) start at w_off:
//   forward  wf[c / 32][t][j][c % 32] = W[t ci + c][j] (first layer: [j][k],
//            k < kpad, zero for k >= 9 ci);
//   dgrad    wd[j / 32][t][c][j % 32] = W[(8 - t) ci + c][j] (mirrored taps):
// what a block reads for a chunk of 32 input channels is contiguous per tap.  A
// thread makes eight consecutive values; neighbours read neighbouring j.
__global__ void __launch_bounds__(256) k_prep_weights(const float* __restrict__ w, ConvTable tab,
                                                      __bf16* __restrict__ wf,
                                                      __bf16* __restrict__ wd) {
  const ConvDesc L = tab.l[blockIdx.y];
  const int nf = L.co * L.kpad / 8, nd = L.has_dgrad ? 9 * L.ci * L.co / 8 : 0;
  const bool first = L.ci % 32 != 0;
  typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
  const float* W = w + L.w_off;
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < nf + nd; e += gridDim.x * blockDim.x) {
    bf16x8 v;
    if (e < nf && first) {
      const int j = 8 * e / L.kpad, k = 8 * e % L.kpad;
      for (int i = 0; i < 8; ++i)
        v[i] = k + i < 9 * L.ci ? (__bf16)W[(int64_t)(k + i) * L.co + j] : (__bf16)0.f;
      *reinterpret_cast<bf16x8*>(wf + L.wf_off + 8 * (int64_t)e) = v;
    } else if (e < nf) {
      const int j = e % L.co, g = e / L.co;  // g = (c / 32 9 + t) 4 + c % 32 / 8
      const int part = g & 3, t = (g >> 2) % 9, cc = (g >> 2) / 9;
      const float* from = W + (int64_t)(t * L.ci + cc * 32 + part * 8) * L.co + j;
      for (int i = 0; i < 8; ++i) v[i] = (__bf16)from[(int64_t)i * L.co];
      *reinterpret_cast<bf16x8*>(wf + L.wf_off + ((int64_t)(g >> 2) * L.co + j) * 32 + part * 8) = v;
    } else {
      const int f = e - nf, part = f & 3, c = (f >> 2) % L.ci, g = (f >> 2) / L.ci;
      const int t = g % 9, jc = g / 9;
      const float* from = W + (int64_t)((8 - t) * L.ci + c) * L.co + jc * 32 + part * 8;
      for (int i = 0; i < 8; ++i) v[i] = (__bf16)from[i];
      *reinterpret_cast<bf16x8*>(wd + L.wd_off + 8 * (int64_t)f) = v;
    }
  }
}

// Dihedral transform of a side x side map: destination pixel (i, j) reads
// source pixel T_f(i, j), f in 0..7: transpose if f & 1, then mirror rows if
// f & 2 and columns if f & 4.
__device__ __forceinline__ int dihedral_src(int i, int j, int f, int side) {
  if (f & 1) {
    const int t = i;
    i = j;
    j = t;
  }
  if (f & 2) i = side - 1 - i;
  if (f & 4) j = side - 1 - j;
  return i * side + j;
}

// Training mini-batch: map idx[b] of (x_all [cin channels], own_all, t_all;
// n_all maps) under the dihedral transform tf[b], into slot b of (xb, ob,
// tb); an index outside [0, n_all) gives a zero slot.
__global__ void __launch_bounds__(256) k_gather_batch(
    const float* __restrict__ x_all, const float* __restrict__ own_all,
    const float* __restrict__ t_all, int64_t n_all, int cin, int side,
    const int32_t* __restrict__ idx, const int32_t* __restrict__ tf, int nb,
    float* __restrict__ xb, float* __restrict__ ob, float* __restrict__ tb) {
  const int npx = side * side;
  const int64_t total = (int64_t)nb * npx;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int b = (int)(e / npx), p = (int)(e % npx);
    const int64_t m = idx[b];
    if (m < 0 || m >= n_all) {
      for (int c = 0; c < cin; ++c) xb[e * cin + c] = 0.f;
      ob[e] = 0.f;
      tb[e] = 0.f;
      continue;
    }
    const int64_t src = m * npx + dihedral_src(p / side, p % side, tf[b] & 7, side);
    for (int c = 0; c < cin; ++c) xb[e * cin + c] = x_all[src * cin + c];
    ob[e] = own_all[src];
    tb[e] = t_all[src];
  }
}

// Inference inputs of map b from its scan's cached table feat[b] (cin inputs,
// then the own-visit term, per pixel).
__global__ void __launch_bounds__(256) k_gather_features(const float* const* __restrict__ feat,
                                                         int nb, int cin, int npx,
                                                         float* __restrict__ x,
                                                         float* __restrict__ own) {
  const int64_t total = (int64_t)nb * npx;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int b = (int)(e / npx), p = (int)(e % npx);
    const float* f = feat[b] + (int64_t)p * (cin + 1);
    for (int c = 0; c < cin; ++c) x[e * cin + c] = f[c];
    own[e] = f[cin];
  }
}

// Prediction output: map b, psi = pref[b] (own + exp(y)) in double, written to
// out[b] (npx values).
__global__ void __launch_bounds__(256) k_output(const float* __restrict__ y,
                                                const float* __restrict__ own, int nb, int npx,
                                                const double* __restrict__ pref,
                                                double* const* __restrict__ out) {
  const int64_t total = (int64_t)nb * npx;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int b = (int)(e / npx), p = (int)(e % npx);
    out[b][p] = pref[b] * ((double)own[e] + exp((double)fminf(y[e], 80.0f)));
  }
}

// Training target: the dimensionless map psi / pref (float).
__global__ void __launch_bounds__(256) k_target(const double* __restrict__ psi, int64_t n,
                                                int64_t per_map, const double* __restrict__ pref,
                                                float* __restrict__ t) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x)
    t[e] = (float)(psi[e] / pref[e / per_map]);
}

// Spot check of map b: relative L2 distance between row `row` of pred[b]
// (side x side) and the exact row exact[b side ..]; one wave per map,
// fixed-order sums.
__global__ void __launch_bounds__(64) k_spot(const double* const* __restrict__ pred,
                                             const double* __restrict__ exact, int side, int x0,
                                             int y0, int step, int w, int h,
                                             double* __restrict__ rel) {
  __shared__ double a[64], b[64];
  const int m = blockIdx.x;
  double num = 0.0, den = 0.0;
  for (int c = threadIdx.x; c < w * h; c += 64) {
    const int u = c % w, v = c / w;
    const double e = exact[(int64_t)m * w * h + c];
    const double d = pred[m][(int64_t)(y0 + step * v) * side + x0 + step * u] - e;
    num += d * d;
    den += e * e;
  }
  a[threadIdx.x] = num;
  b[threadIdx.x] = den;
  __syncthreads();
  for (int s = 32; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      a[threadIdx.x] += a[threadIdx.x + s];
      b[threadIdx.x] += b[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) rel[m] = b[0] > 0 ? sqrt(a[0] / b[0]) : (a[0] > 0 ? 1.0 : 0.0);
}

__global__ void __launch_bounds__(256) k_fill(float* __restrict__ x, int64_t n, float v) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x)
    x[e] = v;
}


// ---------------------------------------------------------------------------
static inline unsigned blocks_for(int64_t n) {
  int64_t g = (n + 255) / 256;
  if (g < 1) g = 1;
  if (g > 65536) g = 65536;
  return (unsigned)g;
}

hipError_t rel_l2(const float* y, const float* own, const float* t, int maps, int npx, float anchor,
                  float* dy, double* loss_map, hipStream_t st) {
  hipLaunchKernelGGL(k_rel_l2, dim3(maps), dim3(256), 0, st, y, own, t, npx, 1.0f / (float)maps,
                     anchor, dy, loss_map);
  return hipGetLastError();
}

hipError_t clip_scale(const float* g, int64_t n, float clip, double* partial, float* scale_norm,
                      hipStream_t st) {
  hipLaunchKernelGGL(k_sumsq, dim3(kNormBlocks), dim3(256), 0, st, g, n, partial);
  hipLaunchKernelGGL(k_clip_scale, dim3(1), dim3(kNormBlocks), 0, st, partial, clip, scale_norm);
  return hipGetLastError();
}

hipError_t adam(float* w, float* m, float* v, const float* g, const float* scale, int64_t n,
                float lr, float b1, float b2, float eps, float bc1, float bc2, hipStream_t st) {
  hipLaunchKernelGGL(k_adam, dim3(blocks_for(n)), dim3(256), 0, st, w, m, v, g, scale, n, lr, b1, b2,
                     eps, bc1, bc2);
  return hipGetLastError();
}

hipError_t prep_weights(const float* w, const ConvTable& tab, __bf16* wf, __bf16* wd,
                        hipStream_t st) {
  int64_t most = 0;
  for (int l = 0; l < tab.n; ++l) {
    const ConvDesc& L = tab.l[l];
    const int64_t n = (int64_t)L.co * L.kpad + (L.has_dgrad ? 9LL * L.ci * L.co : 0);
    most = n > most ? n : most;
  }
  hipLaunchKernelGGL(k_prep_weights, dim3(blocks_for(most), tab.n), dim3(256), 0, st, w, tab, wf,
                     wd);
  return hipGetLastError();
}

hipError_t gather_batch(const float* x_all, const float* own_all, const float* t_all,
                        int64_t n_all, int cin, int side, const int32_t* idx, const int32_t* tf,
                        int nb, float* xb, float* ob, float* tb, hipStream_t st) {
  hipLaunchKernelGGL(k_gather_batch, dim3(blocks_for((int64_t)nb * side * side)), dim3(256), 0, st,
                     x_all, own_all, t_all, n_all, cin, side, idx, tf, nb, xb, ob, tb);
  return hipGetLastError();
}

hipError_t gather_features(const float* const* feat, int nb, int cin, int npx, float* x,
                           float* own, hipStream_t st) {
  hipLaunchKernelGGL(k_gather_features, dim3(blocks_for((int64_t)nb * npx)), dim3(256), 0, st,
                     feat, nb, cin, npx, x, own);
  return hipGetLastError();
}

hipError_t output(const float* y, const float* own, int nb, int npx, const double* pref,
                  double* const* out, hipStream_t st) {
  hipLaunchKernelGGL(k_output, dim3(blocks_for((int64_t)nb * npx)), dim3(256), 0, st, y, own, nb,
                     npx, pref, out);
  return hipGetLastError();
}

hipError_t target(const double* psi, int64_t n, int64_t per_map, const double* pref, float* t,
                  hipStream_t st) {
  hipLaunchKernelGGL(k_target, dim3(blocks_for(n)), dim3(256), 0, st, psi, n, per_map, pref, t);
  return hipGetLastError();
}

hipError_t spot(const double* const* pred, const double* exact, int maps, int side, int x0,
                int y0, int step, int w, int h, double* rel, hipStream_t st) {
  hipLaunchKernelGGL(k_spot, dim3(maps), dim3(64), 0, st, pred, exact, side, x0, y0, step, w, h,
                     rel);
  return hipGetLastError();
}

hipError_t fill(float* x, int64_t n, float v, hipStream_t st) {
  hipLaunchKernelGGL(k_fill, dim3(blocks_for(n)), dim3(256), 0, st, x, n, v);
  return hipGetLastError();
}

}  // namespace nn
}  // namespace dd
