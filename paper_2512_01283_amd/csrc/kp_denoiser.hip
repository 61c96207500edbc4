// kp_denoiser.hip -- kernels of the learned Stokes-map denoiser on gfx950.
//
// The network is a small U-Net (3x3 convolutions at widths c1/c2/c3, 2x2 mean
// pooling, 2x nearest upsampling, skip concatenation, a 1x1 head that adds a
// correction to the input's Q and U).  It is not part of the radiative
// transfer method: it post-processes the step-2 Stokes maps.
//
// Tensors are NHWC BF16 (stored as uint16_t) with a per-pixel stride, so a
// concatenation is two producers writing disjoint channel ranges of one
// buffer.  Pixel p = (n H + h) W + w.  Every channel count is a multiple of 8,
// so 8 consecutive channels are one 16-byte load.
//
// Convolutions (kp_conv.hip) are implicit GEMMs on v_mfma_f32_16x16x32_bf16
// (FP32 accumulation).  The GEMM K index is k = kk * cin + c with kk = 3 dy + dx
// the tap and c the input channel; K = 9 cin is zero-padded to a multiple of
// 32 in the packed weights.  A lane's 8 consecutive K elements never straddle
// a tap because cin % 8 == 0.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "kp_dn_device.hpp"
#include "kp_dn_internal.hpp"

namespace kp {
namespace dn {

// ---------------------------------------------------------------------------
// resampling, 8 channels per thread.  Sizes: fine grid H x W, coarse H/2 x W/2.
// ---------------------------------------------------------------------------
// y (coarse) = mean of each 2x2 block of x (fine)
__global__ void k_pool(const uint16_t* __restrict__ x, int xs, uint16_t* __restrict__ y, int ys, int B, int H, int W,
                       int C) {
  const int Ho = H / 2, Wo = W / 2, C8 = C / 8;
  const size_t n = (size_t)B * Ho * Wo * C8;
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) {
    const int c = (int)(k % C8) * 8;
    const size_t q = k / C8;
    const int w = (int)(q % Wo), h = (int)((q / Wo) % Ho), b = (int)(q / ((size_t)Wo * Ho));
    const size_t f = (size_t)(b * H + 2 * h) * W + 2 * w;
    float s[8], t[8];
    unpack8(ld16(x + f * xs + c), s);
    const size_t nb[3] = {f + 1, f + W, f + W + 1};
    for (int m = 0; m < 3; ++m) {
      unpack8(ld16(x + nb[m] * xs + c), t);
#pragma unroll
      for (int j = 0; j < 8; ++j) s[j] += t[j];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) s[j] *= 0.25f;
    st16(y + q * ys + c, pack8(s));
  }
}

// y (fine) = x (coarse) repeated over each 2x2 block
__global__ void k_up(const uint16_t* __restrict__ x, int xs, uint16_t* __restrict__ y, int ys, int B, int H, int W,
                     int C) {
  const int C8 = C / 8, Wc = W / 2, Hc = H / 2;
  const size_t n = (size_t)B * H * W * C8;
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) {
    const int c = (int)(k % C8) * 8;
    const size_t p = k / C8;
    const int w = (int)(p % W), h = (int)((p / W) % H), b = (int)(p / ((size_t)W * H));
    const size_t q = (size_t)(b * Hc + h / 2) * Wc + w / 2;
    st16(y + p * ys + c, ld16(x + q * xs + c));
  }
}

// gx (coarse) = (sum of each 2x2 block of gy (fine)) where mask (coarse) > 0, else 0
__global__ void k_up_bwd(const uint16_t* __restrict__ gy, int gys, uint16_t* __restrict__ gx, int gxs,
                         const uint16_t* __restrict__ mask, int ms, int B, int H, int W, int C) {
  const int Ho = H / 2, Wo = W / 2, C8 = C / 8;
  const size_t n = (size_t)B * Ho * Wo * C8;
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) {
    const int c = (int)(k % C8) * 8;
    const size_t q = k / C8;
    const int w = (int)(q % Wo), h = (int)((q / Wo) % Ho), b = (int)(q / ((size_t)Wo * Ho));
    const size_t f = (size_t)(b * H + 2 * h) * W + 2 * w;
    float s[8], t[8];
    unpack8(ld16(gy + f * gys + c), s);
    const size_t nb[3] = {f + 1, f + W, f + W + 1};
    for (int m = 0; m < 3; ++m) {
      unpack8(ld16(gy + nb[m] * gys + c), t);
#pragma unroll
      for (int j = 0; j < 8; ++j) s[j] += t[j];
    }
    const u32x4 mv = ld16(mask + q * ms + c);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint16_t mb = (uint16_t)((mv[j / 2] >> (16 * (j & 1))) & 0xFFFFu);
      if (!bf_pos(mb)) s[j] = 0.f;
    }
    st16(gx + q * gxs + c, pack8(s));
  }
}

// dst (fine) = (a (fine) + g (coarse parent) / 4) where mask (fine) > 0, else 0
__global__ void k_pool_bwd_add(const uint16_t* __restrict__ a, int as, const uint16_t* __restrict__ g, int gs,
                               const uint16_t* __restrict__ mask, int ms, uint16_t* __restrict__ dst, int ds, int B,
                               int H, int W, int C) {
  const int C8 = C / 8, Wc = W / 2, Hc = H / 2;
  const size_t n = (size_t)B * H * W * C8;
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) {
    const int c = (int)(k % C8) * 8;
    const size_t p = k / C8;
    const int w = (int)(p % W), h = (int)((p / W) % H), b = (int)(p / ((size_t)W * H));
    const size_t q = (size_t)(b * Hc + h / 2) * Wc + w / 2;
    float s[8], t[8];
    unpack8(ld16(a + p * as + c), s);
    unpack8(ld16(g + q * gs + c), t);
    const u32x4 mv = ld16(mask + p * ms + c);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint16_t mb = (uint16_t)((mv[j / 2] >> (16 * (j & 1))) & 0xFFFFu);
      s[j] = bf_pos(mb) ? s[j] + 0.25f * t[j] : 0.f;
    }
    st16(dst + p * ds + c, pack8(s));
  }
}

// ---------------------------------------------------------------------------
// input normalisation, head, loss, output, optimiser
// ---------------------------------------------------------------------------
// sums[2b] += sum of I, sums[2b+1] += sum of I^2 over image b of maps [B][4][H*W]
// (256-thread blocks; one pair of atomics per block)
__global__ void k_sums(const double* __restrict__ maps, int HW, int runs, double* __restrict__ sums) {
  __shared__ double red[2][4];
  const int b = blockIdx.y;
  double a1 = 0.0, a2 = 0.0;
  for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < HW; p += gridDim.x * blockDim.x) {
    const double* m = maps + (size_t)b * 4 * runs * HW + p;
    const double I = runs == 2 ? 0.5 * (m[0] + m[4 * (size_t)HW]) : m[0];
    a1 += I;
    a2 += I * I;
  }
  for (int off = 32; off > 0; off >>= 1) {
    a1 += __shfl_xor(a1, off);
    a2 += __shfl_xor(a2, off);
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = a1;
    red[1][threadIdx.x >> 6] = a2;
  }
  __syncthreads();
  if (threadIdx.x < 2)
    atomicAdd(sums + 2 * b + threadIdx.x,
              red[threadIdx.x][0] + red[threadIdx.x][1] + red[threadIdx.x][2] + red[threadIdx.x][3]);
}

// Input features of pixel p of image b (s = the image's mean I, Ihat = I/s):
//   x[p][0..7] = ln max(Ihat, 1e-6), Q/I, U/I, V/I (0 where I <= 0), 0, 0, 0, 0 (BF16)
//   xq[p] = (Q/I, U/I) and ihat[p] = Ihat in FP32; tgt[p] = (Q, U) of the
//   target maps / s (FP32).
// With runs == 2 an input image is two independent runs A and B ([8][H][W]:
// A's I, Q, U, V, then B's); (I, Q, U, V) above are then their mean, and
// x[p][4..7] = |S_A - S_B| / (2 I) for S = I, Q, U, V (clamped to 1, 0 where
// I <= 0): a one-sample estimate of the mean's per-pixel noise, unchanged by
// swapping the runs and by the dihedral transforms' signs.
// With aug, image b is first transformed by the dihedral element aug[b] =
// r + 4 f: mirror the width axis if f, then r quarter turns (numpy's rot90;
// dihedral_source gives the pixel read); Stokes (Q, U, V) ->
// ((-1)^r Q, (-1)^(r+f) U, (-1)^f V).  Odd r requires H == W.
// Pixel (h, w) of the image T = rot^r(mirror^f(m)) of an H x W image m
// (code = r + 4 f; rot = numpy's rot90 on (H, W), T is W x H for odd r): on
// return (h, w) is the pixel of m it reads and (sq, su, sv) the signs of its
// Q, U, V.  Source in mirror^f(m): r = 1: (w, W-1-h); r = 2: (H-1-h,
// W-1-w); r = 3: (H-1-w, h); then the mirror flips the column.
__device__ __forceinline__ void dihedral_source(int code, int H, int W, int& h, int& w, double& sq, double& su,
                                                double& sv) {
  const int r = code & 3, f = code >> 2;
  const int h0 = h, w0 = w;
  if (r == 1) {
    h = w0;
    w = W - 1 - h0;
  } else if (r == 2) {
    h = H - 1 - h0;
    w = W - 1 - w0;
  } else if (r == 3) {
    h = H - 1 - w0;
    w = h0;
  }
  if (f) w = W - 1 - w;
  sq = (r & 1) ? -1.0 : 1.0;
  su = ((r + f) & 1) ? -1.0 : 1.0;
  sv = f ? -1.0 : 1.0;
}

__global__ void k_prep(const double* __restrict__ maps, const double* __restrict__ target,
                       const double* __restrict__ sums, const int32_t* __restrict__ aug, int B, int H, int W,
                       int runs, uint16_t* __restrict__ x, float* __restrict__ xq, float* __restrict__ ihat,
                       float* __restrict__ tgt) {
  const int HW = H * W;
  const size_t n = (size_t)B * HW;
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) {
    const size_t b = k / HW;
    int h = (int)(k % HW) / W, w = (int)(k % HW) % W;
    double sq = 1.0, su = 1.0, sv = 1.0;
    if (aug) dihedral_source(aug[b], H, W, h, w, sq, su, sv);
    const size_t p = (size_t)h * W + w;
    const double mean = sums[2 * b] / HW;
    const double* m = maps + b * 4 * runs * HW + p;
    const size_t rb = 4 * (size_t)HW;  // run B's maps (runs == 2)
    auto stokes = [&](int c) { return runs == 2 ? 0.5 * (m[c * (size_t)HW] + m[rb + c * (size_t)HW]) : m[c * (size_t)HW]; };
    const double I = stokes(0);
    const double Ih = mean > 0.0 ? I / mean : 0.0;
    // ratios by division (in the wings of a thick disk I can be subnormal,
    // where 1 / I overflows), clamped to [-1, 1], the range of a physical
    // Stokes vector (I >= |(Q, U, V)|)
    const bool pos = I > 0.0;
    auto frac = [&](double x) { return pos ? (float)fmin(1.0, fmax(-1.0, x / I)) : 0.f; };
    float f8[8];
    f8[0] = (float)log(fmax(Ih, 1e-6));
    f8[1] = (float)sq * frac(stokes(1));
    f8[2] = (float)su * frac(stokes(2));
    f8[3] = (float)sv * frac(stokes(3));
#pragma unroll
    for (int c = 0; c < 4; ++c)
      f8[4 + c] = runs == 2 ? frac(0.5 * fabs(m[c * (size_t)HW] - m[rb + c * (size_t)HW])) : 0.f;
    st16(x + k * 8, pack8(f8));
    xq[2 * k] = f8[1];
    xq[2 * k + 1] = f8[2];
    ihat[k] = (float)Ih;
    if (target) {
      const double* r = target + b * 4 * HW + p;
      const double is = mean > 0.0 ? 1.0 / mean : 0.0;
      tgt[2 * k] = (float)(sq * r[HW] * is);
      tgt[2 * k + 1] = (float)(su * r[2 * (size_t)HW] * is);
    }
  }
}

// Features of the images transformed by `code`, from those of the images as
// they are: the pixel dihedral_source names, with the signs of Q, U and V
// (their BF16 sign bits) flipped as it says.  An averaged inference prepares
// its features once and turns them (5 us for eight 256^2 maps, where forming
// them again took 18 and their sums 11).
__global__ void k_turn(const uint16_t* __restrict__ x, int B, int H, int W, int code, uint16_t* __restrict__ y) {
  const int HW = H * W;
  const size_t n = (size_t)B * HW;
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) {
    const size_t b = k / HW;
    int h = (int)(k % HW) / W, w = (int)(k % HW) % W;
    double sq, su, sv;
    dihedral_source(code, H, W, h, w, sq, su, sv);
    u32x4 v = ld16(x + (b * HW + (size_t)h * W + w) * 8);
    if (sq < 0.0) v[0] ^= 0x80000000u;
    if (su < 0.0) v[1] ^= 0x8000u;
    if (sv < 0.0) v[1] ^= 0x80000000u;
    st16(y + k * 8, v);
  }
}

// out[p][o] = xq[p][o] + hb[o] + sum_c d[p][c] hw[o][c]   (C % 8 == 0)
// Eight lanes per pixel: lane g of a group reads channels 8g + 64i (16 bytes
// each), so a group's loads of one pixel are contiguous and each load
// instruction of a wave reads eight whole pixels (with one lane per pixel
// every instruction touched 64 lines for 16 bytes of each: 3.5x slower).
// The partial sums meet by lane shuffles inside the group; all eight lanes
// of a group take the same p, so a shuffle never reads an inactive lane.
// With TURN the pixels are those of images transformed by `code`, xq belongs
// to the images as they are, and the fractions (q', u') go back to their source
// pixels with the inverse signs (the signs are their own inverses): out[src],
// in the original pixel order, is set if first and added to otherwise.  The
// transform is a bijection of each image's pixels: no two groups write the
// same element.
template <bool TURN>
__global__ void k_head(const uint16_t* __restrict__ d, int C, const float* __restrict__ hw,
                       const float* __restrict__ hb, const float* __restrict__ xq, float* __restrict__ out, int B,
                       int H, int W, int code, int first) {
  const int g = threadIdx.x & 7, HW = H * W;
  const size_t P = (size_t)B * HW;
  const size_t stride = ((size_t)gridDim.x * blockDim.x) >> 3;
  for (size_t p = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) >> 3; p < P; p += stride) {
    float a0 = 0.f, a1 = 0.f;
    for (int c = 8 * g; c < C; c += 64) {
      float v[8];
      unpack8(ld16(d + p * C + c), v);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        a0 += v[j] * hw[c + j];
        a1 += v[j] * hw[C + c + j];
      }
    }
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) {
      a0 += __shfl_xor(a0, off);
      a1 += __shfl_xor(a1, off);
    }
    if (g == 0) {
      if constexpr (TURN) {
        const size_t b = p / HW;
        int h = (int)(p % HW) / W, w = (int)(p % HW) % W;
        double dq, du, dv;
        dihedral_source(code, H, W, h, w, dq, du, dv);
        const float sq = (float)dq, su = (float)du;
        const size_t src = b * HW + (size_t)h * W + w;
        const float q = sq * (sq * xq[2 * src] + hb[0] + a0), u = su * (su * xq[2 * src + 1] + hb[1] + a1);
        out[2 * src] = first ? q : out[2 * src] + q;
        out[2 * src + 1] = first ? u : out[2 * src + 1] + u;
      } else {
        out[2 * p] = xq[2 * p] + hb[0] + a0;
        out[2 * p + 1] = xq[2 * p + 1] + hb[1] + a1;
      }
    }
  }
}

// Relative-error loss: with e = out * Ihat - tgt (both channels) and
// W_b = sum_p Ihat^2 = (sum I^2) / s^2 of image b,
//   loss += sum_p |e|^2 / (B W_b)   (FP64),   go = 2 e Ihat / (B W_b).
// Grid (blocks, B) of 256-thread blocks: image b = blockIdx.y, so the scale
// is formed once per thread; one atomic per block.
__global__ void k_loss(const float* __restrict__ out, const float* __restrict__ tgt,
                       const float* __restrict__ ihat, const double* __restrict__ sums, int B, int HW,
                       float* __restrict__ go, double* __restrict__ loss) {
  __shared__ double red[4];
  const int b = blockIdx.y;
  const double mean = sums[2 * b] / HW;
  const double wb = mean > 0.0 ? sums[2 * b + 1] / (mean * mean) : 0.0;
  const double scale = wb > 0.0 ? 1.0 / (B * wb) : 0.0;
  const float s2 = (float)(2.0 * scale);
  double acc = 0.0;
  for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < HW; p += gridDim.x * blockDim.x) {
    const size_t k = (size_t)b * HW + p;
    const float ih = ihat[k];
    const float2 o = *(const float2*)(out + 2 * k), t = *(const float2*)(tgt + 2 * k);
    const float e0 = o.x * ih - t.x, e1 = o.y * ih - t.y;
    *(float2*)(go + 2 * k) = float2{s2 * e0 * ih, s2 * e1 * ih};
    acc += (double)e0 * e0 + (double)e1 * e1;
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(loss, (red[0] + red[1] + red[2] + red[3]) * scale);
}

// Head backward over a chunk of pixels (256-thread blocks): thread t owns
// channels 8 (t % C8) .. +7 (C8 = C / 8) of pixels t / C8, + 256 / C8, ...:
// ghw[o][c] += sum_p go[p][o] d[p][c]; ghb[o] += sum_p go[p][o];
// gd[p][c] = (sum_o go[p][o] hw[o][c]) where d[p][c] > 0, else 0.
// Per-thread sums are combined in LDS, then one atomic per weight per block.
constexpr int HB_CHUNK = 1024;  // pixels per block
__global__ void k_head_bwd(const float* __restrict__ go, const uint16_t* __restrict__ d, int C,
                           const float* __restrict__ hw, float* __restrict__ ghw, float* __restrict__ ghb,
                           uint16_t* __restrict__ gd, size_t P) {
  __shared__ float red[2 * 512 + 2];
  const int tid = threadIdx.x;
  const int C8 = C >> 3, pp = 256 / C8;
  for (int k = tid; k < 2 * C + 2; k += 256) red[k] = 0.f;
  __syncthreads();
  const int g = tid % C8, pl = tid / C8;
  if (pl < pp) {
    float h0[8], h1[8], a0[8], a1[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      h0[j] = hw[8 * g + j];
      h1[j] = hw[C + 8 * g + j];
      a0[j] = a1[j] = 0.f;
    }
    float sb0 = 0.f, sb1 = 0.f;
    const size_t p0 = (size_t)blockIdx.x * HB_CHUNK;
    const size_t pe = P - p0 < (size_t)HB_CHUNK ? P : p0 + HB_CHUNK;
    for (size_t p = p0 + pl; p < pe; p += pp) {
      const float2 o = *(const float2*)(go + 2 * p);
      float v[8], r[8];
      unpack8(ld16(d + p * C + 8 * g), v);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        a0[j] += o.x * v[j];
        a1[j] += o.y * v[j];
        r[j] = v[j] > 0.f ? o.x * h0[j] + o.y * h1[j] : 0.f;
      }
      st16(gd + p * C + 8 * g, pack8(r));
      sb0 += o.x;
      sb1 += o.y;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      atomicAdd(&red[8 * g + j], a0[j]);
      atomicAdd(&red[C + 8 * g + j], a1[j]);
    }
    if (g == 0) {
      atomicAdd(&red[2 * C], sb0);
      atomicAdd(&red[2 * C + 1], sb1);
    }
  }
  __syncthreads();
  for (int k = tid; k < 2 * C; k += 256) atomicAdd(ghw + k, red[k]);
  if (tid < 2) atomicAdd(ghb + tid, red[2 * C + tid]);
}

// denoised maps: I and V from the input (the two runs' mean if runs == 2),
// Q = scale q' I and U = scale u' I
__global__ void k_output(const double* __restrict__ maps, const float* __restrict__ out, int B, int HW, int runs,
                         double scale, double* __restrict__ dst) {
  const size_t n = (size_t)B * HW;
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) {
    const size_t b = k / HW, p = k % HW;
    const double* m = maps + b * 4 * runs * HW + p;
    double* o = dst + b * 4 * HW + p;
    const size_t rb = 4 * (size_t)HW;
    const double I = runs == 2 ? 0.5 * (m[0] + m[rb]) : m[0];
    o[0] = I;
    o[HW] = (double)out[2 * k] * scale * I;
    o[2 * (size_t)HW] = (double)out[2 * k + 1] * scale * I;
    o[3 * (size_t)HW] = runs == 2 ? 0.5 * (m[3 * (size_t)HW] + m[rb + 3 * (size_t)HW]) : m[3 * (size_t)HW];
  }
}

// (1 - beta) is passed from the host, formed in FP64: 0.999 is not an FP32
// number and 1 - fl(0.999) would be off by 1.3e-5 relative.
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, size_t n, float lr, float b1, float b2, float omb1, float omb2,
                       float eps, float c1, float c2) {
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) {
    const float gk = g[k];
    const float mk = b1 * m[k] + omb1 * gk;
    const float vk = b2 * v[k] + omb2 * gk * gk;
    m[k] = mk;
    v[k] = vk;
    p[k] -= lr * (mk / c1) / (sqrtf(vk / c2) + eps);
  }
}

// FP32 master weights [cout][9][cin_true] -> BF16 GEMM weights
//   w[co][kk * cin + c] (zero for c >= cin_true and for k >= 9 cin, up to kp)
//   wd[ci][kk * cout + co] = w[co][8 - kk][ci] (zero-padded to kpd), if wd != null
__global__ void k_pack(const float* __restrict__ wf, int cout, int cin, int cin_true, int kp, int kpd,
                       uint16_t* __restrict__ w, uint16_t* __restrict__ wd) {
  const size_t n = (size_t)cout * kp;
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) {
    const int co = (int)(k / kp), kx = (int)(k % kp);
    const int kk = kx / cin, c = kx % cin;
    const float v = (kk < 9 && c < cin_true) ? wf[((size_t)co * 9 + kk) * cin_true + c] : 0.f;
    w[k] = f2bf(v);
  }
  if (!wd) return;
  const size_t nd = (size_t)cin_true * kpd;
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < nd; k += (size_t)gridDim.x * blockDim.x) {
    const int ci = (int)(k / kpd), kx = (int)(k % kpd);
    const int kk = kx / cout, co = kx % cout;
    const float v = kk < 9 ? wf[((size_t)co * 9 + (8 - kk)) * cin_true + ci] : 0.f;
    wd[k] = f2bf(v);
  }
}

__global__ void k_zero32(uint32_t* __restrict__ p, size_t n) {
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) p[k] = 0u;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static inline unsigned grid_for(size_t n, size_t cap = 65536) {
  size_t g = (n + 255) / 256;
  if (g > cap) g = cap;
  return (unsigned)(g ? g : 1);
}

void pool(const uint16_t* x, int xs, uint16_t* y, int ys, int B, int H, int W, int C, hipStream_t s) {
  hipLaunchKernelGGL(k_pool, dim3(grid_for((size_t)B * H * W * C / 32)), dim3(256), 0, s, x, xs, y, ys, B, H, W, C);
}
void up(const uint16_t* x, int xs, uint16_t* y, int ys, int B, int H, int W, int C, hipStream_t s) {
  hipLaunchKernelGGL(k_up, dim3(grid_for((size_t)B * H * W * C / 8)), dim3(256), 0, s, x, xs, y, ys, B, H, W, C);
}
void up_bwd(const uint16_t* gy, int gys, uint16_t* gx, int gxs, const uint16_t* mask, int ms, int B, int H, int W,
            int C, hipStream_t s) {
  hipLaunchKernelGGL(k_up_bwd, dim3(grid_for((size_t)B * H * W * C / 32)), dim3(256), 0, s, gy, gys, gx, gxs, mask,
                     ms, B, H, W, C);
}
void pool_bwd_add(const uint16_t* a, int as, const uint16_t* g, int gs, const uint16_t* mask, int ms, uint16_t* dst,
                  int ds, int B, int H, int W, int C, hipStream_t s) {
  hipLaunchKernelGGL(k_pool_bwd_add, dim3(grid_for((size_t)B * H * W * C / 8)), dim3(256), 0, s, a, as, g, gs, mask,
                     ms, dst, ds, B, H, W, C);
}
void sums(const double* maps, int B, int HW, int runs, double* sum, hipStream_t s) {
  hipLaunchKernelGGL(k_sums, dim3(grid_for(HW, 32), B), dim3(256), 0, s, maps, HW, runs, sum);
}
void prep(const double* maps, const double* target, const double* sum, const int32_t* aug, int B, int H, int W,
          int runs, uint16_t* x, float* xq, float* ihat, float* tgt, hipStream_t s) {
  hipLaunchKernelGGL(k_prep, dim3(grid_for((size_t)B * H * W)), dim3(256), 0, s, maps, target, sum, aug, B,
                     H, W, runs, x, xq, ihat, tgt);
}
void turn(const uint16_t* x, int B, int H, int W, int code, uint16_t* y, hipStream_t s) {
  hipLaunchKernelGGL(k_turn, dim3(grid_for((size_t)B * H * W)), dim3(256), 0, s, x, B, H, W, code, y);
}
void head(const uint16_t* d, int C, const float* hw, const float* hb, const float* xq, float* out, int B, int H, int W,
          int code, bool first, hipStream_t s) {
  const dim3 grid(grid_for((size_t)B * H * W * 8));
  if (code < 0) hipLaunchKernelGGL(k_head<false>, grid, dim3(256), 0, s, d, C, hw, hb, xq, out, B, H, W, 0, 1);
  else hipLaunchKernelGGL(k_head<true>, grid, dim3(256), 0, s, d, C, hw, hb, xq, out, B, H, W, code, (int)first);
}
void loss(const float* out, const float* tgt, const float* ihat, const double* sum, int B, int HW, float* go,
          double* l, hipStream_t s) {
  // few blocks per image: the per-block results meet in one FP64 atomic
  hipLaunchKernelGGL(k_loss, dim3(grid_for(HW, 32), B), dim3(256), 0, s, out, tgt, ihat, sum, B, HW, go, l);
}
void head_bwd(const float* go, const uint16_t* d, int C, const float* hw, float* ghw, float* ghb, uint16_t* gd,
              size_t P, hipStream_t s) {
  hipLaunchKernelGGL(k_head_bwd, dim3((unsigned)((P + HB_CHUNK - 1) / HB_CHUNK)), dim3(256), 0, s, go, d, C, hw, ghw,
                     ghb, gd, P);
}
void output(const double* maps, const float* out, int B, int HW, int runs, double scale, double* dst,
            hipStream_t s) {
  hipLaunchKernelGGL(k_output, dim3(grid_for((size_t)B * HW)), dim3(256), 0, s, maps, out, B, HW, runs, scale, dst);
}
void adam(float* p, const float* g, float* m, float* v, size_t n, float lr, int t, hipStream_t s) {
  const double b1 = 0.9, b2 = 0.999;
  const float c1 = (float)(1.0 - std::pow(b1, t)), c2 = (float)(1.0 - std::pow(b2, t));
  hipLaunchKernelGGL(k_adam, dim3(grid_for(n)), dim3(256), 0, s, p, g, m, v, n, lr, (float)b1, (float)b2,
                     (float)(1.0 - b1), (float)(1.0 - b2), 1e-8f, c1, c2);
}
void pack(const float* wf, int cout, int cin, int cin_true, int kp, int kpd, uint16_t* w, uint16_t* wd,
          hipStream_t s) {
  hipLaunchKernelGGL(k_pack, dim3(grid_for((size_t)cout * kp)), dim3(256), 0, s, wf, cout, cin, cin_true, kp, kpd, w,
                     wd);
}
void zero(void* p, size_t bytes, hipStream_t s) {
  hipLaunchKernelGGL(k_zero32, dim3(grid_for(bytes / 4)), dim3(256), 0, s, (uint32_t*)p, bytes / 4);
}

}  // namespace dn
}  // namespace kp
