// unet_wgrad.hip -- the weight gradient of the surrogate's convolutions and the
// backward pass of its activations, for gfx950.
//
// Weight gradient.  dW[tap][c][j] = sum_m x[m + tap][c] dZ[m][j] over the pixels
// m of all images: for each of the nine taps a matrix product whose inner
// index is the pixel, on v_mfma_f32_16x16x32_bf16.  k_wgrad: a block owns 32
// input channels, 32 output channels and all nine taps for a share of the
// 256-pixel tiles.  Per tile it stages the input pixels with a one-pixel halo
// (once, for all taps; the geometry of k_conv_halo) and the tile's dZ in LDS,
// in their NHWC layout, and reads both operands transposed (four pixels of a
// channel per lane) with ds_read_b64_tr_b16, so that nothing is rearranged on
// the way and a tap is an address offset.  Wave w takes channels 16 (w % 2) ..
// +15 and pixels 128 (w / 2) .. +127: 18 MFMAs per 22 LDS reads and 32 pixels.
// The next tile's loads are in flight during the MFMAs.  Each block writes its
// partial sums; k_sum_parts adds the blocks' in a fixed order.
//
// Against im2col in HBM, a GEMM that loaded its operands element by element
// and a reduction pass per layer, the weight gradients of 32 maps (43 GFLOP)
// went from 2.6 ms (im2col 1.2, GEMM 0.8, sums 0.5) to 0.23 (0.18 and 0.05).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "unet_kernels.h"

namespace dd {
namespace nn {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int TP = 256;     // pixels per tile
constexpr int HPMAX = 400;  // halo pixels: 6 x 66, 10 x 34, 18 x 18 or 4 x 10 x 10
constexpr int LD = 40;      // LDS row: 32 channels + 8 padding (BF16)

__device__ __forceinline__ s16x4 tr_read(const __bf16* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4*)const_cast<__bf16*>(p));
}

// MFMA operand of 16 channels x 32 pixels from LDS rows of LD: lane l gets
// channel l % 16 of pixels 8 (l / 16) .. + 7, p being the row of pixel 8 (l / 16) +
// (l % 16) / 4 at channel 4 (l % 4).
__device__ __forceinline__ bf16x8 tr_operand(const __bf16* p) {
  union {
    s16x4 h[2];
    bf16x8 v;
  } u;
  u.h[0] = tr_read(p);
  u.h[1] = tr_read(p + 4 * LD);
  return u.v;
}

struct WgradArgs {
  const __bf16* x;   // input [M][ci], or the skip map [M][ci - c1]
  const __bf16* xc;  // coarse map [M / 4][c1], or NULL
  int c1;
  const __bf16* dz;  // [M][co]
  int M, ci, co, tiles;
  float* part;       // [gridDim.x][9 ci][co]
};

template <bool UPCAT, int LG>
__global__ void __launch_bounds__(256) k_wgrad(WgradArgs p) {
  constexpr int W = 1 << LG;
  constexpr int lgR = LG >= 4 ? 8 - LG : LG, R = 1 << lgR, lgRW = lgR + LG;
  constexpr int HW2 = W + 2, slice = (R + 2) * HW2, HP = (TP >> lgRW) * slice;
  constexpr int XS = (HP * 4 + 255) / 256, ZS = TP * 4 / 256;
  constexpr int kRed = 2 * 18 * 64;  // f32x4 of the cross-wave sum
  constexpr int kTile = (HPMAX + TP) * LD * (int)sizeof(__bf16);
  static_assert(kRed * 16 <= kTile, "the cross-wave sum reuses the tile's LDS");
  __shared__ __attribute__((aligned(16))) unsigned char lds[kTile];
  __bf16* const As = reinterpret_cast<__bf16*>(lds);
  __bf16* const Ds = As + HPMAX * LD;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int jblocks = p.co >> 5;
  const int c0 = (int)(blockIdx.y / jblocks) * 32, j0 = (int)(blockIdx.y % jblocks) * 32;
  const int t0 = (int)((int64_t)p.tiles * blockIdx.x / gridDim.x);
  const int t1 = (int)((int64_t)p.tiles * (blockIdx.x + 1) / gridDim.x);

  bf16x8 xr[XS], zr[ZS];
  auto fetch = [&](int t) {
    const int m0 = t * TP, img0 = m0 >> (2 * LG), y0 = (m0 >> LG) & (W - 1);
#pragma unroll
    for (int i = 0; i < XS; ++i) {
      const int idx = tid + 256 * i, px = idx >> 2, q = idx & 3;
      xr[i] = bf16x8{};
      if (px >= HP) continue;
      const int g = px / slice, rem = px - g * slice;
      const int hr = rem / HW2, hc = rem - hr * HW2;
      const int yy = y0 + hr - 1, xx = hc - 1;
      const int m = (((img0 + g) << LG) + yy) * W + xx;
      if (yy < 0 || yy >= W || xx < 0 || xx >= W || m >= p.M) continue;
      const __bf16* from;
      if (UPCAT && c0 < p.c1) {
        const int sc = ((((img0 + g) << (LG - 1)) + (yy >> 1)) << (LG - 1)) + (xx >> 1);
        from = p.xc + (int64_t)sc * p.c1 + c0 + 8 * q;
      } else if (UPCAT) {
        from = p.x + (int64_t)m * (p.ci - p.c1) + (c0 - p.c1) + 8 * q;
      } else {
        from = p.x + (int64_t)m * p.ci + c0 + 8 * q;
      }
      xr[i] = *reinterpret_cast<const bf16x8*>(from);
    }
#pragma unroll
    for (int i = 0; i < ZS; ++i) {
      const int idx = tid + 256 * i, m = m0 + (idx >> 2), q = idx & 3;
      zr[i] = bf16x8{};
      if (m < p.M) zr[i] = *reinterpret_cast<const bf16x8*>(p.dz + (int64_t)m * p.co + j0 + 8 * q);
    }
  };

  f32x4 acc[9][2];
#pragma unroll
  for (int k = 0; k < 9; ++k) acc[k][0] = acc[k][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int ch = wave & 1, ph = wave >> 1, g = lane >> 4, row = (lane & 15) >> 2;
  const int col = 4 * (lane & 3);
  if (t0 < t1) fetch(t0);
  for (int t = t0; t < t1; ++t) {
    __syncthreads();  // the previous tile is no longer read
#pragma unroll
    for (int i = 0; i < XS; ++i) {
      const int idx = tid + 256 * i;
      if ((idx >> 2) < HP) *reinterpret_cast<bf16x8*>(As + (idx >> 2) * LD + 8 * (idx & 3)) = xr[i];
    }
#pragma unroll
    for (int i = 0; i < ZS; ++i) {
      const int idx = tid + 256 * i;
      *reinterpret_cast<bf16x8*>(Ds + (idx >> 2) * LD + 8 * (idx & 3)) = zr[i];
    }
    __syncthreads();
    if (t + 1 < t1) fetch(t + 1);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int o = ph * 128 + ks * 32 + 8 * g;  // eight pixels of one image row
      const int hb = (o >> lgRW) * slice + ((o >> LG) & (R - 1)) * HW2 + (o & (W - 1));
      const __bf16* za = Ds + (o + row) * LD + col;
      const bf16x8 z0 = tr_operand(za), z1 = tr_operand(za + 16);
      const __bf16* xa = As + (hb + row) * LD + ch * 16 + col;
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        const bf16x8 a = tr_operand(xa + ((tap / 3) * HW2 + tap % 3) * LD);
        acc[tap][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, z0, acc[tap][0], 0, 0, 0);
        acc[tap][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, z1, acc[tap][1], 0, 0, 0);
      }
    }
  }
  // the two pixel halves' sums, then rows c = c0 + 16 ch + 4 (lane / 16) + v,
  // columns j = j0 + 16 jf + lane % 16
  __syncthreads();
  f32x4* red = reinterpret_cast<f32x4*>(lds) + ch * 18 * 64 + lane;
  if (ph == 1) {
#pragma unroll
    for (int k = 0; k < 18; ++k) red[k * 64] = acc[k >> 1][k & 1];
  }
  __syncthreads();
  if (ph == 1) return;
  float* out = p.part + (int64_t)blockIdx.x * 9 * p.ci * p.co;
#pragma unroll
  for (int tap = 0; tap < 9; ++tap)
#pragma unroll
    for (int jf = 0; jf < 2; ++jf) {
      const f32x4 s = acc[tap][jf] + red[(2 * tap + jf) * 64];
      const int c = tap * p.ci + c0 + 16 * ch + 4 * g, j = j0 + 16 * jf + (lane & 15);
#pragma unroll
      for (int v = 0; v < 4; ++v) out[(int64_t)(c + v) * p.co + j] = s[v];
    }
}

// First layer (CI input channels in FP32, 64-pixel rows, 32 output channels):
// the tile's rows of 9 CI values (k = tap CI + c, rounded to BF16, padded to 48)
// are assembled in LDS and read transposed like the channels above; wave w
// takes pixels 64 w .. + 63.
template <int CI>
__global__ void __launch_bounds__(256) k_wgrad_first(const float* __restrict__ x,
                                                     const __bf16* __restrict__ dz, int M,
                                                     int tiles, float* __restrict__ part) {
  constexpr int LG = 6, W = 64, HW2 = W + 2, HP = 6 * HW2, K = 9 * CI, LK = 56;
  static_assert(K <= 48 && LK % 8 == 0, "rows of at most 48 values");
  __shared__ float Xs[HP][CI];
  __shared__ __attribute__((aligned(16))) __bf16 As[TP * LK];
  __shared__ __attribute__((aligned(16))) __bf16 Ds[TP * LD];
  __shared__ f32x4 red[3][6][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4;
  const int row = (lane & 15) >> 2, col = 4 * (lane & 3);
  const int t0 = (int)((int64_t)tiles * blockIdx.x / gridDim.x);
  const int t1 = (int)((int64_t)tiles * (blockIdx.x + 1) / gridDim.x);
  f32x4 acc[3][2];
#pragma unroll
  for (int k = 0; k < 3; ++k) acc[k][0] = acc[k][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int t = t0; t < t1; ++t) {
    const int m0 = t * TP, img0 = m0 >> (2 * LG), y0 = (m0 >> LG) & (W - 1);
    __syncthreads();
    for (int px = tid; px < HP; px += 256) {
      const int hr = px / HW2, hc = px - hr * HW2, yy = y0 + hr - 1, xx = hc - 1;
      const int64_t m = (((int64_t)img0 << LG) + yy) * W + xx;
      const bool in = yy >= 0 && yy < W && xx >= 0 && xx < W && m < M;
#pragma unroll
      for (int c = 0; c < CI; ++c) Xs[px][c] = in ? x[m * CI + c] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < TP * 4 / 256; ++i) {
      const int idx = tid + 256 * i, m = m0 + (idx >> 2), q = idx & 3;
      bf16x8 z{};
      if (m < M) z = *reinterpret_cast<const bf16x8*>(dz + (int64_t)m * 32 + 8 * q);
      *reinterpret_cast<bf16x8*>(Ds + (idx >> 2) * LD + 8 * q) = z;
    }
    __syncthreads();
    {
      const int hb = (tid >> LG) * HW2 + (tid & (W - 1));
      __bf16 v[48];
#pragma unroll
      for (int tap = 0; tap < 9; ++tap)
#pragma unroll
        for (int c = 0; c < CI; ++c)
          v[tap * CI + c] = (__bf16)Xs[hb + (tap / 3) * HW2 + tap % 3][c];
#pragma unroll
      for (int k = K; k < 48; ++k) v[k] = (__bf16)0.f;
#pragma unroll
      for (int q = 0; q < 6; ++q) {
        bf16x8 b;
#pragma unroll
        for (int e = 0; e < 8; ++e) b[e] = v[8 * q + e];
        *reinterpret_cast<bf16x8*>(As + tid * LK + 8 * q) = b;
      }
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int o = wave * 64 + ks * 32 + 8 * g;
      const __bf16* za = Ds + (o + row) * LD + col;
      const bf16x8 z0 = tr_operand(za), z1 = tr_operand(za + 16);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const __bf16* xa = As + (o + row) * LK + 16 * k + col;
        union {
          s16x4 h[2];
          bf16x8 v;
        } u;
        u.h[0] = tr_read(xa);
        u.h[1] = tr_read(xa + 4 * LK);
        acc[k][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(u.v, z0, acc[k][0], 0, 0, 0);
        acc[k][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(u.v, z1, acc[k][1], 0, 0, 0);
      }
    }
  }
  if (wave > 0) {
#pragma unroll
    for (int k = 0; k < 6; ++k) red[wave - 1][k][lane] = acc[k >> 1][k & 1];
  }
  __syncthreads();
  if (wave > 0) return;
  float* out = part + (int64_t)blockIdx.x * K * 32;
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int jf = 0; jf < 2; ++jf) {
      const f32x4 s = ((acc[k][jf] + red[0][2 * k + jf][lane]) + red[1][2 * k + jf][lane]) +
                      red[2][2 * k + jf][lane];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 16 * k + 4 * g + v;
        if (r < K) out[r * 32 + 16 * jf + (lane & 15)] = s[v];
      }
    }
}

// ---------------------------------------------------------------------------
// Backward of an activation: dZ = dA SiLU'(Z), rounded to BF16 (the operand of
// the weight- and data-gradient MFMAs), with the per-channel sums of dZ (the
// bias gradient, from the unrounded values).  dA by mode:
//   plain  the data gradient of the layer that reads this activation;
//   head   dy[m] w[c] (the 1x1 output head), with the head's own sums
//          sum_m dy[m] a[m][c] and sum_m dy[m];
//   up     the four pixels of the nearest-2x upsampling that this coarse pixel
//          became in the concatenation dcat [4 M][ct];
//   pool   the skip channels ct - C .. of dcat [M][ct] plus a quarter of the
//          pooled map's gradient dp [M / 4][C].
// Thread: four channels of one pixel per pass.  Each block writes its sums
// (C, or 2 C + 1 with the head).
enum { ACT_PLAIN = 0, ACT_HEAD = 1, ACT_UP = 2, ACT_POOL = 3 };

struct ActArgs {
  const float* da;    // plain: dA; up, pool: dcat
  const float* dp;    // pool
  int ct;             // up, pool: channels of dcat
  const float* dy;    // head
  const float* hw;    // head weights
  const __bf16* a;    // head: the stored activation
  const float* z;     // pre-activation [M][C]
  int64_t M;
  int lg, C;          // log2 of this map's side, channels
  __bf16* dz;         // [M][C]
  float* part;        // [gridDim.x][C (2 C + 1)]
};

__device__ __forceinline__ float silu_grad(float z) {
  const float s = 1.0f / (1.0f + __expf(-z));
  return s * (1.0f + z * (1.0f - s));
}

template <int MODE>
__global__ void __launch_bounds__(256) k_act_bwd(ActArgs p) {
  __shared__ f32x4 red[2][256];
  __shared__ float red1[256];
  const int tid = threadIdx.x, C = p.C, tpp = C >> 2;  // threads per pixel
  const int c = 4 * (tid & (tpp - 1)), sub = tid / tpp, ppb = 256 / tpp;
  f32x4 bs{0.f, 0.f, 0.f, 0.f}, ws{0.f, 0.f, 0.f, 0.f}, hw{0.f, 0.f, 0.f, 0.f};
  float ds = 0.f;
  if (MODE == ACT_HEAD) hw = *reinterpret_cast<const f32x4*>(p.hw + c);
  const int W = 1 << p.lg;
  for (int64_t m = (int64_t)blockIdx.x * ppb + sub; m < p.M; m += (int64_t)gridDim.x * ppb) {
    const int64_t e = m * C + c;
    f32x4 da;
    if (MODE == ACT_PLAIN) {
      da = *reinterpret_cast<const f32x4*>(p.da + e);
    } else if (MODE == ACT_HEAD) {
      const float d = p.dy[m];
      da = f32x4{d * hw[0], d * hw[1], d * hw[2], d * hw[3]};
      const bf16x4 a = *reinterpret_cast<const bf16x4*>(p.a + e);
#pragma unroll
      for (int k = 0; k < 4; ++k) ws[k] = __builtin_fmaf(d, (float)a[k], ws[k]);
      ds += d;
    } else {
      const int xx = (int)(m & (W - 1)), yy = (int)((m >> p.lg) & (W - 1));
      const int64_t n = m >> (2 * p.lg);
      if (MODE == ACT_UP) {
        const int64_t b = (((n * 2 * W + 2 * yy) * 2 * W) + 2 * xx) * p.ct + c;
        auto at = [&](int64_t i) { return *reinterpret_cast<const f32x4*>(p.da + i); };
        const int64_t dn = (int64_t)2 * W * p.ct;
        da = at(b) + at(b + p.ct) + at(b + dn) + at(b + dn + p.ct);
      } else {
        const int64_t q = ((n * (W / 2) + yy / 2) * (W / 2) + xx / 2) * C + c;
        da = *reinterpret_cast<const f32x4*>(p.da + m * p.ct + (p.ct - C) + c);
        const f32x4 dp = *reinterpret_cast<const f32x4*>(p.dp + q);
#pragma unroll
        for (int k = 0; k < 4; ++k) da[k] += 0.25f * dp[k];
      }
    }
    const f32x4 z = *reinterpret_cast<const f32x4*>(p.z + e);
    bf16x4 o;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float v = da[k] * silu_grad(z[k]);
      o[k] = (__bf16)v;
      bs[k] += v;
    }
    *reinterpret_cast<bf16x4*>(p.dz + e) = o;
  }
  // the block's sums over its pixels, in a fixed order
  red[0][tid] = bs;
  if (MODE == ACT_HEAD) {
    red[1][tid] = ws;
    red1[tid] = ds;
  }
  __syncthreads();
  for (int s = ppb >> 1; s > 0; s >>= 1) {
    if (sub < s) {
      red[0][tid] += red[0][tid + s * tpp];
      if (MODE == ACT_HEAD) {
        red[1][tid] += red[1][tid + s * tpp];
        red1[tid] += red1[tid + s * tpp];
      }
    }
    __syncthreads();
  }
  if (sub != 0) return;
  const int len = MODE == ACT_HEAD ? 2 * C + 1 : C;
  float* out = p.part + (int64_t)blockIdx.x * len;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    out[c + k] = red[0][tid][k];
    if (MODE == ACT_HEAD) out[C + c + k] = red[1][tid][k];
  }
  if (MODE == ACT_HEAD && c == 0) out[2 * C] = red1[0];
}

// Sums of partial results over blocks, in a fixed order: out[e] = sum_s part[s
// stride + e].  A block takes 256 / G consecutive outputs of one entry, G
// threads each (thread g adds parts g, g + G, ...): 16 for the long sums, whose
// chains of loads would otherwise outlast the rest of the launch, else 4.
// Blocks are dealt to the entries in order, `first` being an entry's first one.
constexpr int sum_groups(int splits) { return splits > 32 ? 16 : 4; }

template <int G>
__device__ __forceinline__ void sum_part(const PartDesc& d, float* red) {
  constexpr int E = 256 / G;
  const int i = threadIdx.x % E, g = threadIdx.x / E;
  const int64_t e = (int64_t)((int)blockIdx.x - d.first) * E + i;
  float s = 0.f;
  if (e < d.n) {
#pragma unroll 8
    for (int k = g; k < d.splits; k += G) s += d.part[(int64_t)k * d.stride + e];
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = G / 2; h > 0; h >>= 1) {
    if (g < h) red[threadIdx.x] += red[threadIdx.x + h * E];
    __syncthreads();
  }
  if (g == 0 && e < d.n) d.out[e] = red[i];
}

__global__ void __launch_bounds__(256) k_sum_parts(PartTable tab) {
  __shared__ float red[256];
  int y = 0;  // the last entry whose first block is not past this one
  for (int hi = tab.n - 1; y < hi;) {
    const int mid = (y + hi + 1) >> 1;
    if (tab.l[mid].first <= (int)blockIdx.x)
      y = mid;
    else
      hi = mid - 1;
  }
  const PartDesc d = tab.l[y];
  if (sum_groups(d.splits) == 16)
    sum_part<16>(d, red);
  else
    sum_part<4>(d, red);
}

hipError_t launch_act(int mode, const ActArgs& p, hipStream_t st) {
  const dim3 grid(kActBlocks);
  if (p.C < 32 || p.C > 256 || (p.C & (p.C - 1)) != 0 || p.M <= 0) return hipErrorInvalidValue;
  switch (mode) {
    case ACT_PLAIN: hipLaunchKernelGGL(k_act_bwd<ACT_PLAIN>, grid, dim3(256), 0, st, p); break;
    case ACT_HEAD: hipLaunchKernelGGL(k_act_bwd<ACT_HEAD>, grid, dim3(256), 0, st, p); break;
    case ACT_UP: hipLaunchKernelGGL(k_act_bwd<ACT_UP>, grid, dim3(256), 0, st, p); break;
    default: hipLaunchKernelGGL(k_act_bwd<ACT_POOL>, grid, dim3(256), 0, st, p); break;
  }
  return hipGetLastError();
}

}  // namespace

// Blocks sharing a layer's tiles: one per CU in all, at most one per tile.  (Two
// per CU took the same time and doubled the partial sums, 245 instead of 122 MB
// for the network.)
int wgrad_splits(int64_t M, int ci, int co) {
  const int64_t tiles = (M + TP - 1) / TP;
  const int64_t grid = ci % 32 == 0 ? (ci / 32) * (int64_t)(co / 32) : 1;
  return (int)std::max<int64_t>(1, std::min<int64_t>({tiles, 256 / grid, 256}));
}

hipError_t wgrad(const __bf16* x, const __bf16* coarse, int c1, const __bf16* dz, int B, int lg,
                 int ci, int co, float* part, hipStream_t st) {
  const int64_t M = (int64_t)B << (2 * lg);
  if (M <= 0 || M > (1ll << 30) || ci % 32 != 0 || co % 32 != 0 || (coarse && (c1 % 32 != 0 || lg < 4)))
    return hipErrorInvalidValue;
  WgradArgs p{x, coarse, c1, dz, (int)M, ci, co, (int)((M + TP - 1) / TP), part};
  const dim3 grid(wgrad_splits(M, ci, co), (ci / 32) * (co / 32));
#define DD_WGRAD(LG)                                                                    \
  case LG:                                                                              \
    if (coarse)                                                                         \
      hipLaunchKernelGGL((k_wgrad<true, LG>), grid, dim3(256), 0, st, p);               \
    else                                                                                \
      hipLaunchKernelGGL((k_wgrad<false, LG>), grid, dim3(256), 0, st, p);              \
    break;
  switch (lg) {
    DD_WGRAD(3) DD_WGRAD(4) DD_WGRAD(5) DD_WGRAD(6)
    default: return hipErrorInvalidValue;
  }
#undef DD_WGRAD
  return hipGetLastError();
}

hipError_t wgrad_first(const float* x, const __bf16* dz, int B, int ci, float* part,
                       hipStream_t st) {
  const int64_t M = (int64_t)B << 12;
  if (M <= 0 || M > (1ll << 30) || ci != 5) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_wgrad_first<5>, dim3(wgrad_splits(M, ci, 32)), dim3(256), 0, st, x, dz,
                     (int)M, (int)(M / TP), part);
  return hipGetLastError();
}

hipError_t act_bwd(const float* da, const float* z, int64_t M, int C, __bf16* dz, float* part,
                   hipStream_t st) {
  return launch_act(ACT_PLAIN, ActArgs{da, nullptr, 0, nullptr, nullptr, nullptr, z, M, 0, C, dz, part},
                    st);
}
hipError_t act_bwd_head(const float* dy, const float* hw, const __bf16* a, const float* z, int64_t M,
                        int C, __bf16* dz, float* part, hipStream_t st) {
  return launch_act(ACT_HEAD, ActArgs{nullptr, nullptr, 0, dy, hw, a, z, M, 0, C, dz, part}, st);
}
hipError_t act_bwd_up(const float* dcat, int ct, const float* z, int B, int lg, int C, __bf16* dz,
                      float* part, hipStream_t st) {
  return launch_act(ACT_UP, ActArgs{dcat, nullptr, ct, nullptr, nullptr, nullptr, z,
                                    (int64_t)B << (2 * lg), lg, C, dz, part}, st);
}
hipError_t act_bwd_pool(const float* dcat, int ct, const float* dp, const float* z, int B, int lg,
                        int C, __bf16* dz, float* part, hipStream_t st) {
  return launch_act(ACT_POOL, ActArgs{dcat, dp, ct, nullptr, nullptr, nullptr, z,
                                      (int64_t)B << (2 * lg), lg, C, dz, part}, st);
}

hipError_t sum_parts(PartTable tab, hipStream_t st) {
  if (tab.n <= 0) return hipSuccess;
  int64_t blocks = 0;
  for (int k = 0; k < tab.n; ++k) {
    tab.l[k].first = (int)blocks;
    const int per = 256 / sum_groups(tab.l[k].splits);
    blocks += (tab.l[k].n + per - 1) / per;
  }
  hipLaunchKernelGGL(k_sum_parts, dim3((unsigned)blocks), dim3(256), 0, st, tab);
  return hipGetLastError();
}

}  // namespace nn
}  // namespace dd
