// unet_kernels.h -- launchers of the surrogate's HIP kernels (unet_conv.hip,
// unet_wgrad.hip, unet_kernels.hip).  All activations are NHWC FP32; GEMM operands BF16.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace dd {
namespace nn {

// One convolution layer for the weight-layout kernel.
struct ConvDesc {
  int ci, co, kpad, has_dgrad;  // kpad: forward weights per output channel (>= 9 ci)
  int64_t w_off, wf_off, wd_off;  // FP32 master, BF16 forward and dgrad (k_prep_weights)
};
constexpr int kMaxConv = 16;
struct ConvTable {
  int n;
  ConvDesc l[kMaxConv];
};
constexpr int kNormBlocks = 256;  // partial sums of the gradient norm

// 3x3 convolutions (unet_conv.hip) of x [B][side][side][ci], side = 2^lg in
// 8..64, weights wt [ci / 32][tap][co][32] (k_prep_weights):
//   conv3_silu:        z = conv + bias, act = SiLU(z) (z stored when non-NULL;
//                      with pool non-NULL, side >= 16, also the 2x2 average of
//                      act, [B][side/2][side/2][co]: the four BF16 values in row order, x 0.25,
//                      rounded to BF16);
//   conv3_upcat_silu:  the same on the channel concatenation [nearest-2x
//                      upsampling of coarse [B][side/2][side/2][c1], skip
//                      [B][side][side][c2]];
//   conv3_silu_head:   co = 32, then y = SiLU(z) . head[0..31] + head[32]
//                      (act and z stored when non-NULL);
//   conv3_plain:       out = conv in FP32 (the data gradient, with the dgrad layout);
//   conv3_first_silu:  ci < 32 with 9 ci <= 64, co = 32, weights [32][64].
// ci, c1 and co must be multiples of 32 except in conv3_first_silu.
hipError_t conv3_silu(const __bf16* x, int B, int lg, int ci, const __bf16* wt, const float* bias,
                      __bf16* act, float* z, int co, __bf16* pool, hipStream_t st);
hipError_t conv3_upcat_silu(const __bf16* coarse, int c1, const __bf16* skip, int c2, int B,
                            int lg, const __bf16* wt, const float* bias, __bf16* act, float* z,
                            int co, hipStream_t st);
hipError_t conv3_silu_head(const __bf16* x, int B, int lg, int ci, const __bf16* wt,
                           const float* bias, const float* head, __bf16* act, float* z, float* y,
                           hipStream_t st);
hipError_t conv3_plain(const __bf16* x, int B, int lg, int ci, const __bf16* wt, float* out, int co,
                       hipStream_t st);
hipError_t conv3_first_silu(const float* x, int B, int lg, int ci, const __bf16* wt,
                            const float* bias, __bf16* act, float* z, hipStream_t st);

// Weight gradient (unet_wgrad.hip) of a 3x3 convolution of x [B][side][side][ci]
// (or the concatenation of the upsampled coarse map, c1 channels, and the skip
// map x) for dz [B][side][side][co]: wgrad_splits() partial sums [9 ci][co]
// each.  wgrad_first: the first layer (ci = 5, co = 32, side 64, x FP32).
int wgrad_splits(int64_t M, int ci, int co);
hipError_t wgrad(const __bf16* x, const __bf16* coarse, int c1, const __bf16* dz, int B, int lg,
                 int ci, int co, float* part, hipStream_t st);
hipError_t wgrad_first(const float* x, const __bf16* dz, int B, int ci, float* part,
                       hipStream_t st);
// dZ = dA SiLU'(z) as BF16 and its kActBlocks partial channel sums (see
// k_act_bwd): dA the data gradient itself, dy w (head; 2 C + 1 sums per
// block: bias, head weights, head bias), the upsampling's adjoint on the
// first channels of dcat, or the skip channels of dcat and the pooling's
// adjoint of dp.
constexpr int kActBlocks = 512;
hipError_t act_bwd(const float* da, const float* z, int64_t M, int C, __bf16* dz, float* part,
                   hipStream_t st);
hipError_t act_bwd_head(const float* dy, const float* hw, const __bf16* a, const float* z, int64_t M,
                        int C, __bf16* dz, float* part, hipStream_t st);
hipError_t act_bwd_up(const float* dcat, int ct, const float* z, int B, int lg, int C, __bf16* dz,
                      float* part, hipStream_t st);
hipError_t act_bwd_pool(const float* dcat, int ct, const float* dp, const float* z, int B, int lg,
                        int C, __bf16* dz, float* part, hipStream_t st);
// out[e] = sum over s < splits of part[s stride + e], e < n, for every entry.
struct PartDesc {
  const float* part;
  int64_t stride, n;
  int splits;
  float* out;
  int first = 0;  // set by sum_parts
};
struct PartTable {
  int n;
  PartDesc l[2 * kMaxConv + 1];
};
hipError_t sum_parts(PartTable tab, hipStream_t st);
// Squared relative L2 error per map (loss_map[b]) of prediction own + exp(y)
// against t; dy of the mean over maps of that error plus the anchor term
// (anchor / npx) sum (r/t)^2 (y - ln r)^2, r = max(t - own, 1e-6 t).
hipError_t rel_l2(const float* y, const float* own, const float* t, int maps, int npx, float anchor,
                  float* dy, double* loss_map, hipStream_t st);
// scale_norm[0] = clipping factor of g (global norm), scale_norm[1] = |g|;
// partial holds kNormBlocks doubles.
hipError_t clip_scale(const float* g, int64_t n, float clip, double* partial, float* scale_norm,
                      hipStream_t st);
hipError_t adam(float* w, float* m, float* v, const float* g, const float* scale, int64_t n,
                float lr, float b1, float b2, float eps, float bc1, float bc2, hipStream_t st);
hipError_t prep_weights(const float* w, const ConvTable& tab, __bf16* wf, __bf16* wd,
                        hipStream_t st);
hipError_t gather_batch(const float* x_all, const float* own_all, const float* t_all,
                        int64_t n_all, int cin, int side, const int32_t* idx, const int32_t* tf,
                        int nb, float* xb, float* ob, float* tb, hipStream_t st);
hipError_t gather_features(const float* const* feat, int nb, int cin, int npx, float* x,
                           float* own, hipStream_t st);
hipError_t output(const float* y, const float* own, int nb, int npx, const double* pref,
                  double* const* out, hipStream_t st);
hipError_t target(const double* psi, int64_t n, int64_t per_map, const double* pref, float* t,
                  hipStream_t st);
// Relative L2 error per map of the predicted values on the probe sub-grid
// (x0 + step u, y0 + step v), u < w, v < h, of side x side maps against the
// exact values exact[map][v w + u].
hipError_t spot(const double* const* pred, const double* exact, int maps, int side, int x0,
                int y0, int step, int w, int h, double* rel, hipStream_t st);
hipError_t fill(float* x, int64_t n, float v, hipStream_t st);

}  // namespace nn
}  // namespace dd
