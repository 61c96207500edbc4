// kp_conv.hip -- the denoiser's 3x3 convolutions (forward and input gradient).
//
// Implicit GEMMs on v_mfma_f32_16x16x32_bf16 with FP32 accumulation over NHWC
// BF16 tensors; every channel count is a multiple of 8.  Two kernels: k_conv3
// for images of a few hundred pixels, k_conv3_tile for the rest.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <utility>

#include "kp_conv_rule.hpp"
#include "kp_dn_device.hpp"
#include "kp_dn_internal.hpp"

namespace kp {
namespace dn {

// ---------------------------------------------------------------------------
// 3x3 convolution as an implicit GEMM:
//   y[p][n] = epi( sum_{kk, c} x[p + off(kk)][c] * w[n][kk * cin + c] )
// off(kk) = (kk / 3 - 1, kk % 3 - 1), zero outside the image.  The forward
// pass uses the layer's weights; the input gradient of a layer uses the same
// kernel with the flipped, transposed weights wd[ci][kk * cout + co] =
// w[co][8 - kk][ci], because off(8 - kk) = -off(kk).
// One wave computes 32 pixels x 64 output channels (2 x 4 MFMA tiles).
// ---------------------------------------------------------------------------
// MODE: CONV_RELU (bias, relu), CONV_PLAIN (neither), CONV_MASK (zero where mask <= 0)
template <int MODE>
__global__ void __launch_bounds__(256) k_conv3(ConvArgs a) {
  const int lane = threadIdx.x & 63;
  const int wave = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int P = a.B * a.H * a.W;
  const int ngroups = (a.nout + 63) >> 6;
  const int ptile = wave / ngroups, ng = wave - ptile * ngroups;
  if (ptile * 32 >= P) return;
  const int i = lane & 15, g = lane >> 4;
  int ph[2], pw[2], pn[2];
  bool pv[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int p = ptile * 32 + 16 * r + i;
    pv[r] = p < P;
    const int q = pv[r] ? p : 0;
    pw[r] = q % a.W;
    ph[r] = (q / a.W) % a.H;
    pn[r] = q / (a.W * a.H);
  }
  const int n0 = ng * 64;
  const int ntile = min(4, (a.nout - n0) >> 4);
  f32x4 acc[2][4];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[r][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  const uint16_t* wrow[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) wrow[t] = a.w + (size_t)(n0 + 16 * min(t, ntile - 1) + i) * a.kp + 8 * g;
  const int K = 9 * a.cin;
  int kk = 0, c = 8 * g;
  while (c >= a.cin) {
    c -= a.cin;
    ++kk;
  }
  const u32x4 zero = {0u, 0u, 0u, 0u};
  for (int k0 = 0; k0 < K; k0 += 32) {
    const int dy = kk / 3 - 1, dx = kk % 3 - 1;
    u32x4 av[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int hh = ph[r] + dy, ww = pw[r] + dx;
      const bool ok = pv[r] && kk < 9 && hh >= 0 && hh < a.H && ww >= 0 && ww < a.W;
      av[r] = ok ? ld16(a.x + ((size_t)(pn[r] * a.H + hh) * a.W + ww) * a.xs + c) : zero;
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (t < ntile) {
        const u32x4 bv = ld16(wrow[t] + k0);
        acc[0][t] = mfma(av[0], bv, acc[0][t]);
        acc[1][t] = mfma(av[1], bv, acc[1][t]);
      }
    }
    c += 32;
    while (c >= a.cin) {
      c -= a.cin;
      ++kk;
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    if (t >= ntile) continue;
    const int n = n0 + 16 * t + i;
    const float bn = MODE == CONV_RELU ? a.bias[n] : 0.f;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int p = ptile * 32 + 16 * r + 4 * g + j;
        if (p >= P) continue;
        float v = acc[r][t][j] + bn;
        if (MODE == CONV_RELU) v = fmaxf(v, 0.f);
        if (MODE == CONV_MASK && !bf_pos(a.mask[(size_t)p * a.ms + n])) v = 0.f;
        a.y[(size_t)p * a.ys + n] = f2bf(v);
      }
  }
}

// ---------------------------------------------------------------------------
// The same convolution from LDS.  A workgroup of WR x WC waves owns a tile of
// WR RW rows x 16 columns of one image and 16 NT WC output channels; a wave
// computes RW rows x 16 NT of the channels (RW x NT MFMA tiles; the operands
// are weights x pixels, so a lane ends with 4 NT consecutive channels of one
// pixel and stores them at once).  The K loop runs over blocks of 32 input
// channels, the nine taps inside: every output adds up in the same order
// whatever the tile.
//
// What bounds it is how much else a wave has to issue between MFMAs, so
// little is left in the loop:
// - Halo and weights go from memory to LDS by LDS DMA (buffer loads that
//   write LDS), double buffered and issued a group at a time among the first
//   five taps' MFMAs; pixels outside the image and channels past cin take an
//   offset past the resource's range, which loads zero.  No staging registers,
//   no LDS stores, no branches.
// - A pixel row's operand is read once per horizontal tap and kept for the
//   three vertical ones: 3 (RW + 2) operand reads per block, not 9 RW.
// - LDS rows are 64 bytes without padding; chunk c of row or column r sits at
//   slot c ^ 2 ((r >> 2) & 1), free of conflicts under the rule of
//   kp_dn_device.hpp for 16 consecutive rows from any offset.
// - The workgroup stays for all its items: the next item's first block loads
//   during the last taps, and its results are stored while the block after
//   that is computed.  Two waves per SIMD cover each other's epilogue.
// The map below a skip connection is read at half resolution in place (no
// upsampled copy), and the 2x2 means that the next level starts from are
// taken from the rounded outputs in the epilogue.
//
// Measured (8 images, 192 -> 64 channels at 256^2, 115.96 GFLOP): 160 us with
// one tile per workgroup staged through registers, 125 us as LDS DMA with four
// waves of 8 x 4 tiles, 105 us with the addresses kept in registers, 90 us
// (1.29 PFLOP/s) with eight waves of 8 x 2.  64 -> 64: 87 -> 41 us, of which
// 27 us are its 134 MB of maps at the rate of a copy.  Two images of 100 x 172,
// 48 -> 48: 14.3 -> 6.6 us; of 25 x 43, 192 -> 192: 26.5 -> 6.7 us.
// ---------------------------------------------------------------------------
constexpr int CT_RSRC3 = 0x00020000;  // buffer resource word 3: raw 32-bit data
constexpr int CT_OUT = 0x7FFFFFF0;    // an offset past every resource's range
__device__ const u32x4 ct_zero[4] = {};

template <int NT, int RW, int WR, int WC>
struct CtShape {
  static constexpr int ROWS = WR * RW, NW = WR * WC;           // output rows of a tile, waves
  static constexpr int HP = (ROWS + 2) * CT_E;                 // halo pixels
  static constexpr int HI = (HP + 15) / 16, WI = 9 * NT * WC;  // 1 KB pieces (16 rows of 64 bytes): halo, weights
  static constexpr int BUF = (HI + WI) * 1024;
  static constexpr int HU = (HI + NW - 1) / NW, WU = (WI + NW - 1) / NW, NP = HU + WU;  // pieces per wave
  static constexpr int PG = (NP + 5 * NT - 1) / (5 * NT);  // pieces issued per group of RW MFMAs
  static constexpr int LDS = 2 * BUF + 2048;
};

// FAR: tiles whose rows lie more than 2^31 bytes apart from end to end, which
// a buffer's 32-bit offsets cannot reach: the halo loads take full addresses
template <int MODE, int NT, int RW, int WR, int WC, bool FAR>
__device__ __forceinline__ void conv3_tile(const ConvArgs& a) {
  using S = CtShape<NT, RW, WR, WC>;
  constexpr int NTW = NT * WC;  // channel tiles of the workgroup
  __shared__ __attribute__((aligned(1024))) unsigned char lds0[S::BUF];
  __shared__ __attribute__((aligned(1024))) unsigned char lds1[S::BUF];
  __shared__ __attribute__((aligned(16))) float bias[512];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wrow = wv / WC, wcol = wv % WC;
  const int i = lane & 15, g = lane >> 4;
  const int ngroups = a.nout / (16 * NTW);
  const int txn = (a.W + 15) >> 4, tyn = (a.H + S::ROWS - 1) / S::ROWS;
  const int items = a.B * tyn * txn * ngroups, nb = (a.cin + 31) >> 5;
  const int nlow = a.xl ? a.cl >> 5 : 0;  // blocks taken from the half-resolution map
  // workgroups go to the 8 XCDs round-robin: XCD x takes an eighth of the items in a row
  const int xcd = blockIdx.x & 7, stride = gridDim.x >> 3;
  const int last = (int)((long)items * (xcd + 1) >> 3);
  int item = (int)((long)items * xcd >> 3) + (int)(blockIdx.x >> 3);
  if (item >= last) return;
  if (MODE == CONV_RELU)
    for (int n = threadIdx.x; n < a.nout; n += 64 * S::NW) bias[n] = a.bias[n];

  const int slot = lane & 3, prow = lane >> 2;
  auto decode = [&](int it, int& ng, int& tx, int& ty, int& img) CT_INLINE {
    ng = it % ngroups;
    it /= ngroups;
    tx = it % txn;
    it /= txn;
    ty = it % tyn;
    img = it / tyn;
  };
  // 16-byte slot of chunk c of halo column hx / operand row r
  auto swz = [&](int hx, int c) CT_INLINE { return c ^ (((hx >> 2) & 1) << 1); };
  // offsets of this lane's halo chunks from the tile's corner in the current
  // source, CT_OUT outside the image: bytes, or (FAR) pixels
  int hoff[S::HU];
  const uint16_t* xbase = nullptr;
  int xstride = 0;
  __amdgpu_buffer_rsrc_t xr;
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, a.nout * a.kp * 2, CT_RSRC3);
  // weight row i of wave column w's tile t of a tap is channel n0 + 16 NT w + 4 NT (i >> 2) + 4 t + (i & 3)
  const int wlane = ((4 * NT * (prow >> 2) + (prow & 3)) * a.kp + 8 * swz(prow, slot)) * 2;
  int wbase = 0;
  int wpre[S::WU];
  ct_for<S::WU>([&](auto K) CT_INLINE {
    const int n = wv + S::NW * K, tap = n / NTW, t = n % NTW;
    wpre[K] = ((16 * NT * (t / NT) + 4 * (t % NT)) * a.kp + tap * a.cin) * 2;
  });
  unsigned hrag = 0;  // bit u: halo piece u's chunk lies past cin in the last block
  ct_for<S::HU>([&](auto K) CT_INLINE {
    if ((a.cin & 31) && 8 * swz((16 * (wv + S::NW * K) + prow) % CT_E, slot) >= (a.cin & 31)) hrag |= 1u << K;
  });
  auto prep = [&](int it, int cb) CT_INLINE {
    int ng, tx, ty, img;
    decode(it, ng, tx, ty, img);
    const int low = cb < nlow;
    const int y0 = ty * S::ROWS - 1, x0 = tx * 16 - 1;
    const int W = a.W >> low, H = a.H >> low;
    xstride = low ? a.xls : a.xs;
    xbase = (low ? a.xl : a.x) + ((long)(img * H + (y0 >> low)) * W + (x0 >> low)) * xstride;
    xr = __builtin_amdgcn_make_buffer_rsrc((void*)xbase, 0, CT_OUT - 16, CT_RSRC3);
    ct_for<S::HU>([&](auto U) CT_INLINE {
      constexpr int u = U;
      const int hp = 16 * (wv + S::NW * u) + prow;
      const int hy = hp / CT_E, hx = hp - hy * CT_E;
      const int yy = y0 + hy, xx = x0 + hx;
      const bool ok = hp < S::HP && yy >= 0 && yy < a.H && xx >= 0 && xx < a.W;
      const int pix = ((yy >> low) - (y0 >> low)) * W + (xx >> low) - (x0 >> low);
      hoff[u] = !ok ? CT_OUT : FAR ? pix : (pix * xstride + 8 * swz(hx, slot)) * 2;
    });
    wbase = ng * 16 * NTW * a.kp * 2;
  };
  auto leave = [&]() CT_INLINE {
    xr = __builtin_amdgcn_make_buffer_rsrc((void*)xbase, 0, 0, CT_RSRC3);
    if constexpr (FAR) ct_for<S::HU>([&](auto U) CT_INLINE { hoff[U] = CT_OUT; });
  };
  // piece k of a block (byte offset soff = 64 cb, rag = CT_OUT in a partial last block, else 0)
  auto piece = [&](auto K, int soff, int rag, unsigned char* buf) CT_INLINE {
    constexpr int k = K;
    if constexpr (k < S::HU) {
      const int n = wv + S::NW * k;
      if (S::NW * k + S::NW - 1 < S::HI || n < S::HI) {
        auto* dst = (__attribute__((address_space(3))) void*)(buf + n * 1024);
        const int off = hoff[k] | ((int)(hrag << (31 - k)) >> 31 & rag);
        if constexpr (FAR) {
          const uint16_t* src = xbase + (size_t)(uint32_t)off * (uint32_t)xstride + soff / 2 + 8 * swz((16 * n + prow) % CT_E, slot);
          if (off >= CT_OUT) src = (const uint16_t*)ct_zero;
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, dst, 16, 0, 0);
        } else {
          __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, dst, 16, off, soff, 0, 0);
        }
      }
    } else if constexpr (k < S::NP) {
      const int n = wv + S::NW * (k - S::HU);
      if (S::NW * (k - S::HU) + S::NW - 1 < S::WI || n < S::WI)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            wres, (__attribute__((address_space(3))) void*)(buf + (S::HI + n) * 1024), 16, wlane,
            wbase + wpre[k - S::HU] + soff, 0, 0);
    }
  };
  f32x4 acc[RW][NT];
  uint2 mk[RW][NT];
  // operand addresses: pixel column i + dx of halo row RW wv + r + dy, chunk g
  int poff[3];
  ct_for<3>([&](auto D) CT_INLINE { poff[D] = (RW * wrow * CT_E + i + D) * 64 + 16 * swz(i + D, g); });
  const int woff = (S::HI + NT * wcol) * 1024 + i * 64 + 16 * swz(i, g);
  auto get_mask = [&](int it) CT_INLINE {
    int ng, tx, ty, img;
    decode(it, ng, tx, ty, img);
    const int n = ng * 16 * NTW + 16 * NT * wcol + 4 * NT * g;
    const int xx = min(tx * 16 + i, a.W - 1);
    ct_for<RW>([&](auto R) CT_INLINE {
      const int yy = min(ty * S::ROWS + RW * wrow + (int)R, a.H - 1);
      const size_t p = (size_t)(img * a.H + yy) * a.W + xx;
      ct_for<NT>([&](auto T) CT_INLINE { mk[R][T] = *(const uint2*)(a.mask + p * a.ms + n + 4 * T); });
    });
  };
  auto epilogue = [&](int it) CT_INLINE {
    int ng, tx, ty, img;
    decode(it, ng, tx, ty, img);
    const int n = ng * 16 * NTW + 16 * NT * wcol + 4 * NT * g;
    const int xx = tx * 16 + i;
    f32x4 bn[NT];
    if (MODE == CONV_RELU) ct_for<NT>([&](auto T) CT_INLINE { bn[T] = *(const f32x4*)(bias + n + 4 * T); });
    uint2 o[2][NT];  // rows r - 1 (r odd) and r
    ct_for<RW>([&](auto R) CT_INLINE {
      constexpr int r = R;
      const int yy = ty * S::ROWS + RW * wrow + r;
      ct_for<NT>([&](auto T) CT_INLINE {
        constexpr int t = T;
        f32x4 v = acc[r][t];
        if (MODE == CONV_RELU) {
          v += bn[t];
          v = f32x4{fmaxf(v[0], 0.f), fmaxf(v[1], 0.f), fmaxf(v[2], 0.f), fmaxf(v[3], 0.f)};
        }
        if (MODE == CONV_MASK) {
          const uint2 m = mk[r][t];
          if (!bf_pos((uint16_t)m.x)) v[0] = 0.f;
          if (!bf_pos((uint16_t)(m.x >> 16))) v[1] = 0.f;
          if (!bf_pos((uint16_t)m.y)) v[2] = 0.f;
          if (!bf_pos((uint16_t)(m.y >> 16))) v[3] = 0.f;
        }
        o[r & 1][t] = uint2{f2bf2(v[0], v[1]), f2bf2(v[2], v[3])};
      });
      const bool ok = yy < a.H && xx < a.W;
      if (ok) {
        uint16_t* y = a.y + ((size_t)(img * a.H + yy) * a.W + xx) * a.ys + n;
        ct_for<NT>([&](auto T) CT_INLINE { *(uint2*)(y + 4 * T) = o[r & 1][T]; });
      }
      // 2x2 means: the even lane of a pair of columns, rows r - 1 and r
      if constexpr (MODE == CONV_RELU && RW > 1 && (r & 1)) {
        if (a.yp) {
          uint2 m[NT];
          ct_for<NT>([&](auto T) CT_INLINE {
            constexpr int t = T;
            auto mean = [&](uint32_t p0, uint32_t p1) CT_INLINE {  // two channels
              const uint32_t q0 = __builtin_amdgcn_update_dpp(0, p0, 0xB1, 0xF, 0xF, true);
              const uint32_t q1 = __builtin_amdgcn_update_dpp(0, p1, 0xB1, 0xF, 0xF, true);
              auto lo = [](uint32_t w) CT_INLINE { return __uint_as_float(w << 16); };
              auto hi = [](uint32_t w) CT_INLINE { return __uint_as_float(w & 0xFFFF0000u); };
              float s0 = lo(p0) + lo(q0), s1 = hi(p0) + hi(q0);
              s0 += lo(p1);
              s1 += hi(p1);
              s0 += lo(q1);
              s1 += hi(q1);
              return f2bf2(s0 * 0.25f, s1 * 0.25f);
            };
            m[t] = uint2{mean(o[0][t].x, o[1][t].x), mean(o[0][t].y, o[1][t].y)};
          });
          if (ok && !(i & 1)) {
            uint16_t* y = a.yp + ((size_t)(img * (a.H >> 1) + (yy >> 1)) * (a.W >> 1) + (xx >> 1)) * a.yps + n;
            ct_for<NT>([&](auto T) CT_INLINE { *(uint2*)(y + 4 * T) = m[T]; });
          }
        }
      }
    });
  };
  auto clear = [&]() CT_INLINE {
    ct_for<RW>([&](auto R) CT_INLINE {
      ct_for<NT>([&](auto T) CT_INLINE { acc[R][T] = f32x4{0.f, 0.f, 0.f, 0.f}; });
    });
  };
  auto taps = [&](const unsigned char* cur, int soff, int rag, unsigned char* nxt) CT_INLINE {
    u32x4 P[RW + 2][3], wf[NT];
    auto rd_w = [&](auto TAP, auto T) CT_INLINE { wf[T] = *(const u32x4*)(cur + woff + (TAP * NTW + T) * 1024); };
    auto rd_p = [&](auto R, auto DX) CT_INLINE { P[R][DX] = *(const u32x4*)(cur + poff[DX] + R * CT_E * 64); };
    ct_for<NT>([&](auto T) CT_INLINE { rd_w(std::integral_constant<int, 0>{}, T); });
    ct_for<RW>([&](auto R) CT_INLINE { rd_p(R, std::integral_constant<int, 0>{}); });
    ct_for<9>([&](auto TAP) CT_INLINE {
      constexpr int tap = TAP, dy = tap / 3, dx = tap % 3;
      constexpr int ndy = tap < 8 ? (tap + 1) / 3 : 0, ndx = (tap + 1) % 3;  // the next tap
      ct_for<NT>([&](auto T) CT_INLINE {
        constexpr int t = T, q = tap * NT + t;
        if constexpr (q * S::PG < S::NP)
          ct_for<S::PG>([&](auto J) CT_INLINE { piece(std::integral_constant<int, q * S::PG + J>{}, soff, rag, nxt); });
        if constexpr (tap < 2) {  // dy = 0: its rows, shared out over the groups
          constexpr int per = (RW + NT - 1) / NT;
          ct_for<per>([&](auto J) CT_INLINE {
            if constexpr (t * per + J < RW)
              rd_p(std::integral_constant<int, t * per + J>{}, std::integral_constant<int, ndx>{});
          });
        } else if constexpr (tap < 8 && t == 0) {
          rd_p(std::integral_constant<int, ndy ? RW + ndy - 1 : 0>{}, std::integral_constant<int, ndx>{});
        }
        ct_for<RW>([&](auto R) CT_INLINE { acc[R][t] = mfma(wf[t], P[R + dy][dx], acc[R][t]); });
        if constexpr (tap < 8) rd_w(std::integral_constant<int, tap + 1>{}, T);
        __builtin_amdgcn_sched_barrier(0);
      });
    });
  };
  int done = -1;  // the finished item whose outputs are still in acc
  int cb = 0;
  prep(item, 0);
  ct_for<S::NP>([&](auto K) CT_INLINE { piece(K, 0, nb == 1 && (a.cin & 31) ? CT_OUT : 0, lds0); });
  clear();
  auto step = [&](unsigned char* cur, unsigned char* nxt) CT_INLINE -> bool {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // this wave's loads into cur have landed (vmcnt 0)
    __syncthreads();
    const bool end = cb + 1 == nb;
    const int nitem = end ? item + stride : item, ncb = end ? 0 : cb + 1;
    const bool more = nitem < last;
    // past the last item the loads go on and find an empty range (or, FAR, nothing but zeros)
    if (more && (end || ncb == nlow)) prep(nitem, ncb);
    else if (!more) leave();
    if (done >= 0) {
      epilogue(done);
      clear();
      done = -1;
    }
    if (MODE == CONV_MASK && end) get_mask(item);
    taps(cur, ncb * 64, ncb + 1 == nb && (a.cin & 31) ? CT_OUT : 0, nxt);
    if (end) done = item;
    item = nitem;
    cb = ncb;
    return more;
  };
  for (;;) {
    if (!step(lds0, lds1)) break;
    if (!step(lds1, lds0)) break;
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);
  epilogue(done);
}

template <int MODE, int NT, int RW, int WR, int WC, bool FAR>
__global__ void __launch_bounds__(64 * WR * WC) k_conv3_tile(ConvArgs a) {
  conv3_tile<MODE, NT, RW, WR, WC, FAR>(a);
}

// ---------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------
template <int MODE, int NT, int RW, int WR, int WC, bool FAR = false>
static void launch_tile(const ConvArgs& a, hipStream_t s) {
  using S = CtShape<NT, RW, WR, WC>;
  const long items =
      (long)a.B * ((a.H + S::ROWS - 1) / S::ROWS) * ((a.W + 15) / 16) * (a.nout / (16 * NT * WC));
  const long cap = (long)CT_CUS * (160 * 1024 / S::LDS);
  const long grid = std::min((items + 7) / 8 * 8, cap);
  hipLaunchKernelGGL((k_conv3_tile<MODE, NT, RW, WR, WC, FAR>), dim3((unsigned)grid), dim3(64 * S::NW), 0, s, a);
}

template <int MODE>
static void conv3_mode(const ConvArgs& a, hipStream_t s) {
  const size_t P = (size_t)a.B * a.H * a.W;
  if (!conv_tiled(P)) {
    const size_t waves = ((P + 31) / 32) * ((a.nout + 63) / 64);
    hipLaunchKernelGGL(k_conv3<MODE>, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, a);
    return;
  }
  int rows, nt;
  conv_tile_shape(a.B, a.H, a.W, a.cin, a.nout, rows, nt);
  // bytes from a tile's first row to its last
  const bool far = (double)(rows + 2) * a.W * std::max(a.xs, a.xl ? a.xls : 0) * 2.0 >= 2147000000.0;
  switch (far ? -nt : rows * 8 + nt) {
#define KP_TILE(N)                                                          \
  case 32 * 8 + N: launch_tile<MODE, N, 4, 8, 1>(a, s); break;              \
  case 16 * 8 + N: launch_tile<MODE, N, 2, 8, 1>(a, s); break;              \
  case 8 * 8 + N: launch_tile<MODE, N, 2, 4, 1>(a, s); break;               \
  case -N: launch_tile<MODE, N, 2, 4, 1, true>(a, s); break;
    KP_TILE(1) KP_TILE(2) KP_TILE(3)
#undef KP_TILE
    // four channel tiles by 32 rows: two columns of waves with 8 x 2 MFMA
    // tiles read 48 operands per 144 MFMAs, eight waves of 4 x 4 read 54
    // (384 -> 128 channels, 128^2 x 8: 82.6 against 85.0 us); with a mask's
    // registers on top the 4 x 4 tiles fit better
    case 32 * 8 + 4:
      if (MODE == CONV_MASK) launch_tile<MODE, 4, 4, 8, 1>(a, s);
      else launch_tile<MODE, 2, 8, 4, 2>(a, s);
      break;
    case 16 * 8 + 4: launch_tile<MODE, 4, 2, 8, 1>(a, s); break;
    case 8 * 8 + 4: launch_tile<MODE, 4, 2, 4, 1>(a, s); break;
    case -4: launch_tile<MODE, 4, 2, 4, 1, true>(a, s); break;
  }
}

void conv3(const ConvArgs& a, int mode, hipStream_t s) {
  if (mode == CONV_RELU) conv3_mode<CONV_RELU>(a, s);
  else if (mode == CONV_PLAIN) conv3_mode<CONV_PLAIN>(a, s);
  else conv3_mode<CONV_MASK>(a, s);
}

}  // namespace dn
}  // namespace kp
