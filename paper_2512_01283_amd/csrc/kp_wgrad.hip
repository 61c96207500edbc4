// kp_wgrad.hip -- weight and bias gradients of the denoiser's 3x3 convolutions.
//
//   gw[co][kk][c] += sum_p gz[p][co] * x[p + off(kk)][c],   gb[co] += sum_p gz[p][co]
//
// off(kk) = (kk / 3 - 1, kk % 3 - 1), zero outside the image; a contraction
// over pixels on v_mfma_f32_16x16x32_bf16.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <utility>

#include "kp_dn_device.hpp"
#include "kp_dn_internal.hpp"

namespace kp {
namespace dn {

// ---------------------------------------------------------------------------
// One launch takes every layer of a network.  A layer's gradient is cut into
// blocks of 16 MR output channels x 16 G input channels x 9 taps (G = 4, 2 or
// 1, the most that fits what is left), each block's pixels into chunks, one
// workgroup per chunk, so many that all of them together are about one per CU
// and take about the same time.  The partial blocks go to scratch with plain
// stores and k_wgrad_sum adds them up: one block per CU for the whole
// network, where a launch per layer wrote and read 38 MB for each of them.
//
// A workgroup stays for its chunk of tiles of 8 rows x 32 columns.  gz and
// the halo of x go to LDS as they lie in memory (pixel by pixel, 128 bytes
// each) by LDS DMA, double buffered and issued among the MFMAs; the operands,
// which run along pixels, are read with ds_read_b64_tr_b16, which transposes
// 4 pixels x 16 channels on the way, so nothing is transposed by hand.  Eight
// waves: wave w takes input channels 16 (w % G) of the block for all 16 MR
// output channels and nine taps (9 MR accumulators), and RS = G of the 8
// rows.  An x row is read once per horizontal shift and multiplied with the
// three gz rows it meets, which stay in registers: 6 (RS + 2) + 2 RS MR reads
// of 8 bytes per 9 RS MR MFMAs.
//
// What bounds it: a tile of 48 x 64 channels takes 3.4 us, 2.0 of them MFMAs
// at the clock the card holds under them, and 2.4 without its loads.  Eight
// 256^2 maps, widths 48, 96, 192 (263 GFLOP of products, sums included): nine
// launches of 64 x 64 blocks transposed through registers and one of a
// narrower kernel, with their sums, 776 us; here 387 us.  Widths 64, 128, 256:
// 640 us (0.73 PFLOP/s).  Two maps of 100 x 172, widths 48, 96, 192: 54 us.
//
// LDS: the 32-byte segment t (16 channels) of pixel column p sits at segment
// t ^ h(p), h(p) = bit 1 of p + 2 (bit 3 of p): the 32 lanes of a pass read 4
// consecutive pixels and the 4 that lie 8 further on, and their 8 segments
// fall on different banks at every horizontal shift.
// ---------------------------------------------------------------------------
constexpr int WT_ROWS = 8, WT_COLS = 32;             // pixels of a tile
constexpr int WT_E = WT_COLS + 2;                    // halo columns
constexpr int WT_XP = (WT_ROWS + 2) * WT_E;          // halo pixels (340)
constexpr int WT_XI = (WT_XP + 7) / 8;               // 1 KB pieces (8 pixels): halo, gz
constexpr int WT_ZI = WT_ROWS * WT_COLS / 8;
constexpr int WT_BUF = (WT_XI + WT_ZI) * 1024;       // 75 KB
constexpr int WT_XU = (WT_XI + 7) / 8, WT_ZU = WT_ZI / 8;  // pieces per wave
constexpr int WT_RSRC3 = 0x00020000;                 // buffer resource word 3: raw 32-bit data
constexpr int WT_OUT = 0x7FFFFFF0;                   // an offset past every resource's range
__device__ const u32x4 wt_zero[4] = {};

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

__device__ __forceinline__ int wt_swz(int p) { return ((p >> 1) & 1) | (((p >> 3) & 1) << 1); }

// 8 consecutive pixels of 16 channels, transposed: lane (i, g) gets pixels 8g..8g+7 of channel i
__device__ __forceinline__ u32x4 wt_read(const unsigned char* lo, const unsigned char* hi) {
  const uint2 a = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)lo));
  const uint2 b = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)hi));
  return u32x4{a.x, a.y, b.x, b.y};
}

// blocks of k_wgrad_sum for a partial block
__host__ __device__ constexpr int wgrad_sum_blocks(int mr, int g) {
  return (int)((wgrad_block_floats(mr, g) + 1023) / 1024);
}

template <int MR, int G, bool FAR>
__device__ __forceinline__ void wgrad_block(const WgradLayer& a, int m0, int c0, bool first, int t_begin, int t_end,
                                            float* __restrict__ part, unsigned char* lds0, unsigned char* lds1) {
  constexpr int S = 8 / G, RS = WT_ROWS / S;  // row sets, rows of a wave
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = lane & 15, g = lane >> 4;
  const int cg = wv % G, set = wv / G;
  const int tyn = (a.H + WT_ROWS - 1) / WT_ROWS, txn = (a.W + WT_COLS - 1) / WT_COLS;
  const int low = a.low, Ws = a.W >> low, Hs = a.H >> low;

  // loads: piece n holds pixels 8n..8n+7, this lane 16-byte slot lane & 7 of pixel 8n + (lane >> 3)
  const int slot = lane & 7, lpx = lane >> 3;
  auto chunk_of = [&](int p) CT_INLINE { return slot ^ (2 * wt_swz(p)); };  // channels 8 chunk..
  int xrel[WT_XU], xpos[WT_XU];  // offset from the tile's corner; row << 8 | column
  ct_for<WT_XU>([&](auto U) CT_INLINE {
    const int px = 8 * (wv + 8 * U) + lpx, hy = px / WT_E, hx = px - hy * WT_E, ch = chunk_of(hx);
    const int pix = low ? ((hy + 1) >> 1) * Ws + ((hx + 1) >> 1) : hy * Ws + hx;
    const bool ok = px < WT_XP && ch < 2 * G && c0 + 8 * ch < a.cin;
    xrel[U] = !ok ? WT_OUT : FAR ? pix : (pix * a.xs + 8 * ch) * 2;
    xpos[U] = hy << 8 | hx;
  });
  // gz: pieces wv, wv + 8, .. hold a quarter row each, two rows apart
  const int zcol = 8 * (wv & 3) + lpx, zch = chunk_of(zcol);
  const int zpix = (wv >> 2) * a.W + zcol;
  const int zrel = zch >= 2 * MR || m0 + 8 * zch >= a.cout ? WT_OUT : FAR ? zpix : (zpix * a.gzs + 8 * zch) * 2;
  const uint16_t *xb = nullptr, *zb = nullptr;
  __amdgpu_buffer_rsrc_t xr, zr;
  int y0 = 0, x0 = 0;
  auto prep = [&](int t) CT_INLINE {
    const int img = t / (tyn * txn), rt = t - img * tyn * txn;
    y0 = (rt / txn) * WT_ROWS;
    x0 = t < t_end ? (rt % txn) * WT_COLS : a.W + 1;
    xb = a.x + ((long)(img * Hs + (y0 >> low) - 1) * Ws + (x0 >> low) - 1) * a.xs + c0;
    zb = a.gz + ((long)(img * a.H + y0) * a.W + x0) * a.gzs + m0;
    xr = __builtin_amdgcn_make_buffer_rsrc((void*)xb, 0, WT_OUT - 16, WT_RSRC3);
    zr = __builtin_amdgcn_make_buffer_rsrc((void*)zb, 0, WT_OUT - 16, WT_RSRC3);
  };
  auto piece = [&](auto K, unsigned char* buf) CT_INLINE {
    constexpr int k = K;
    constexpr bool is_x = k < WT_XU;
    constexpr int u = is_x ? k : k - WT_XU;
    const int n = wv + 8 * u;
    if (is_x && n >= WT_XI) return;
    auto* dst = (__attribute__((address_space(3))) void*)(buf + (is_x ? n : WT_XI + n) * 1024);
    const int yy = is_x ? y0 - 1 + (xpos[is_x ? u : 0] >> 8) : y0 + (wv >> 2) + 2 * u;
    const int xx = is_x ? x0 - 1 + (xpos[is_x ? u : 0] & 255) : x0 + zcol;
    const int off = (unsigned)yy < (unsigned)a.H && (unsigned)xx < (unsigned)a.W ? (is_x ? xrel[is_x ? u : 0] : zrel) : WT_OUT;
    if constexpr (FAR) {
      const uint16_t* src = is_x ? xb + (size_t)(uint32_t)off * (uint32_t)a.xs + 8 * chunk_of(xpos[is_x ? u : 0] & 255)
                                 : zb + ((size_t)(uint32_t)off + (size_t)2 * u * a.W) * (uint32_t)a.gzs + 8 * zch;
      if (off == WT_OUT) src = (const uint16_t*)wt_zero;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, dst, 16, 0, 0);
    } else if constexpr (is_x) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, dst, 16, off, 0, 0, 0);
    } else {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(zr, dst, 16, off, 4 * u * a.W * a.gzs, 0, 0);
    }
  };
  constexpr int NP = WT_XU + WT_ZU, PG = (NP + RS) / (RS + 1);  // pieces issued per row

  // operands: this lane points at channels 4 (lane & 3).. of pixel 8g + (lane >> 2 & 3) (and 4 further on)
  const int lc = 8 * (lane & 3), lp = 8 * g + ((lane >> 2) & 3);
  int xo[3][2], zo[2];
  ct_for<3>([&](auto D) CT_INLINE {
    ct_for<2>([&](auto H) CT_INLINE {
      const int p = lp + D + 4 * H;
      xo[D][H] = (set * RS * WT_E + p) * 128 + 32 * (cg ^ wt_swz(p)) + lc;
    });
  });
  ct_for<2>([&](auto H) CT_INLINE {  // segment M lies at ^ 32 M
    const int p = lp + 4 * H;
    zo[H] = WT_XI * 1024 + (set * RS * WT_COLS + p) * 128 + 32 * wt_swz(p) + lc;
  });
  f32x4 acc[MR][9];
  ct_for<MR>([&](auto M) CT_INLINE { ct_for<9>([&](auto T) CT_INLINE { acc[M][T] = f32x4{0.f, 0.f, 0.f, 0.f}; }); });
  float bsum[MR];
  ct_for<MR>([&](auto M) CT_INLINE { bsum[M] = 0.f; });
  const bool do_bias = first && cg == 0;

  auto rows = [&](const unsigned char* cur, unsigned char* nxt) CT_INLINE {
    u32x4 A[3][MR];  // gz rows r, r - 1, r - 2
    ct_for<RS + 2>([&](auto R) CT_INLINE {
      constexpr int r = R;
      u32x4 x[3];
      ct_for<3>([&](auto D) CT_INLINE {
        x[D] = wt_read(cur + xo[D][0] + r * WT_E * 128, cur + xo[D][1] + r * WT_E * 128);
      });
      if constexpr (r < RS)
        ct_for<MR>([&](auto M) CT_INLINE {
          A[r % 3][M] = wt_read(cur + (zo[0] ^ (32 * M)) + r * WT_COLS * 128, cur + (zo[1] ^ (32 * M)) + r * WT_COLS * 128);
        });
      ct_for<PG>([&](auto J) CT_INLINE {
        if constexpr (r * PG + J < NP) piece(std::integral_constant<int, r * PG + J>{}, nxt);
      });
      // the oldest gz row first: its products need nothing that was just read of gz
      ct_for<3>([&](auto Q) CT_INLINE {
        constexpr int dy = 2 - Q, y = r - dy;
        if constexpr (y >= 0 && y < RS)
          ct_for<3>([&](auto D) CT_INLINE {
            ct_for<MR>([&](auto M) CT_INLINE { acc[M][3 * dy + D] = mfma(A[y % 3][M], x[D], acc[M][3 * dy + D]); });
          });
      });
      if constexpr (r < RS)
        if (do_bias)
          ct_for<MR>([&](auto M) CT_INLINE {
            float f[8];
            unpack8(A[r % 3][M], f);
            bsum[M] += ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
          });
      __builtin_amdgcn_sched_barrier(0);  // keep later rows' reads from being hoisted (registers)
    });
  };
  int t = t_begin;
  prep(t);
  ct_for<NP>([&](auto K) CT_INLINE { piece(K, lds0); });
  auto step = [&](unsigned char* cur, unsigned char* nxt) CT_INLINE {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // this wave's loads into cur have landed (vmcnt 0)
    __syncthreads();
    prep(++t);  // past the last tile the loads go on and find nothing
    rows(cur, nxt);
  };
  while (t + 2 <= t_end) {
    step(lds0, lds1);
    step(lds1, lds0);
  }
  if (t < t_end) step(lds0, lds1);
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();
  // the row sets' sums meet in LDS, one set after the other: 16 output
  // channels [co][tap][c] of the block after the other, then the biases
  ct_for<MR>([&](auto M) CT_INLINE {
    bsum[M] += __shfl_xor(bsum[M], 16);
    bsum[M] += __shfl_xor(bsum[M], 32);
  });
  // (rows of 144 G + 4 floats: the four co of a store fall on different banks)
  constexpr int NB = 16 * 9 * 16 * G, ROW = 9 * 16 * G + 4;
  static_assert(2 * 16 * ROW * 4 <= WT_BUF && 16 * ROW * 4 + 16 * MR * 4 <= WT_BUF && MR <= 3);
  auto slab = [&](int m) CT_INLINE { return (float*)(m < 2 ? lds0 : lds1) + (m < 2 ? m : 0) * 16 * ROW; };
  float* const bias = (float*)lds1 + 16 * ROW;
  auto merge = [&](auto ADD) CT_INLINE {
    ct_for<MR>([&](auto M) CT_INLINE {
      ct_for<4>([&](auto J) CT_INLINE {
        float* q = slab(M) + (4 * g + J) * ROW + 16 * cg + i;
        float v[9];
        ct_for<9>([&](auto T) CT_INLINE { v[T] = acc[M][T][(int)J]; });
        if constexpr (ADD) ct_for<9>([&](auto T) CT_INLINE { v[T] += q[T * 16 * G]; });
        ct_for<9>([&](auto T) CT_INLINE { q[T * 16 * G] = v[T]; });
        __builtin_amdgcn_sched_barrier(0);  // nine at a time (registers)
      });
      if (do_bias && g == 0) bias[16 * M + i] = ADD ? bias[16 * M + i] + bsum[M] : bsum[M];
    });
  };
  if (set == 0) merge(std::false_type{});
  __syncthreads();
  for (int s = 1; s < S; ++s) {
    if (set == s) merge(std::true_type{});
    __syncthreads();
  }
  ct_for<MR>([&](auto M) CT_INLINE {
    for (int k = 4 * threadIdx.x; k < NB; k += 4 * 512) {
      const int co = k / (9 * 16 * G);
      *(f32x4*)(part + M * NB + k) = *(const f32x4*)(slab(M) + k + 4 * co);
    }
  });
  if (first && threadIdx.x < 16 * MR) part[MR * NB + threadIdx.x] = bias[threadIdx.x];
}

template <int MR, bool FAR>
__global__ void __launch_bounds__(512) k_wgrad(WgradBatch b) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds0[WT_BUF];
  __shared__ __attribute__((aligned(1024))) unsigned char lds1[WT_BUF];
  // the 8 XCDs take workgroups round-robin: regroup so that one XCD runs the
  // blocks of consecutive chunks (they share gz and x in its L2)
  int wg = blockIdx.x;
  if (wg < b.wgs - b.wgs % 8) wg = (wg & 7) * (b.wgs / 8) + (wg >> 3);
  int j = 0;
  while (j + 1 < b.n && wg >= b.l[j + 1].first) ++j;
  const WgradLayer& a = b.l[j];
  wg -= a.first;
  // blocks of the layer by width: class 0 holds 64 input channels, 1 32, 2 16
  int cls = 0, c0 = 0;
  float* part = b.part + a.part;
  for (; cls < 2; ++cls) {
    const int n = a.mt * a.units[cls] * a.nch[cls];
    if (wg < n) break;
    wg -= n;
    c0 += a.units[cls] * (64 >> cls);
    part += (size_t)n * wgrad_block_floats(MR, 4 >> cls);
  }
  const int tiles = a.mt * a.units[cls], chn = wg / tiles, tile = wg - chn * tiles;
  const int m = tile / a.units[cls], u = tile - m * a.units[cls];
  part += (size_t)wg * wgrad_block_floats(MR, 4 >> cls);
  c0 += u * (64 >> cls);
  const int nt = a.B * ((a.H + WT_ROWS - 1) / WT_ROWS) * ((a.W + WT_COLS - 1) / WT_COLS);
  const int t0 = (int)((long)nt * chn / a.nch[cls]), t1 = (int)((long)nt * (chn + 1) / a.nch[cls]);
  const bool first = c0 == 0 && a.gb;
  if (cls == 0) wgrad_block<MR, 4, FAR>(a, 16 * MR * m, c0, first, t0, t1, part, lds0, lds1);
  else if (cls == 1) wgrad_block<MR, 2, FAR>(a, 16 * MR * m, c0, first, t0, t1, part, lds0, lds1);
  else wgrad_block<MR, 1, FAR>(a, 16 * MR * m, c0, first, t0, t1, part, lds0, lds1);
}

// gw, gb += the sums of the partial blocks over their chunks: a thread takes
// four neighbouring floats of a block, 256 threads 1024 of them; eight chunks'
// loads are in flight
template <int MR>
__global__ void __launch_bounds__(256) k_wgrad_sum(WgradBatch b) {
  int j = 0;
  while (j + 1 < b.n && (int)blockIdx.x >= b.l[j + 1].sum_first) ++j;
  const WgradLayer& a = b.l[j];
  int r = blockIdx.x - a.sum_first, cls = 0, c0 = 0;
  const float* part = b.part + a.part;
  for (; cls < 2; ++cls) {
    const int tiles = a.mt * a.units[cls], n = tiles * wgrad_sum_blocks(MR, 4 >> cls);
    if (r < n) break;
    r -= n;
    c0 += a.units[cls] * (64 >> cls);
    part += (size_t)tiles * a.nch[cls] * wgrad_block_floats(MR, 4 >> cls);
  }
  const int G = 4 >> cls, sb = wgrad_sum_blocks(MR, G), tiles = a.mt * a.units[cls];
  const int tile = r / sb, m = tile / a.units[cls];
  c0 += (tile - m * a.units[cls]) * 16 * G;
  const int e = (r - tile * sb) * 1024 + 4 * threadIdx.x, nw = 16 * MR * 9 * 16 * G;
  const bool bias = e >= nw;
  if (e >= nw + (c0 == 0 && a.gb ? 16 * MR : 0)) return;
  const size_t blk = wgrad_block_floats(MR, G), step = tiles * blk;
  part += tile * blk + e;
  f32x4 s[8] = {};
  int k = 0;
  for (; k + 8 <= a.nch[cls]; k += 8)
#pragma unroll
    for (int u = 0; u < 8; ++u) s[u] += *(const f32x4*)(part + (k + u) * step);
  for (; k < a.nch[cls]; ++k) s[0] += *(const f32x4*)(part + k * step);
  const f32x4 t = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
  const int co = 16 * MR * m + (bias ? e - nw : e / (9 * 16 * G));
  const int tap = e / (16 * G) % 9, c = c0 + e % (16 * G);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (bias) a.gb[co + q] += t[q];
    else if (c + q < a.cin_true) a.gw[((size_t)co * 9 + tap) * a.gws + c + q] += t[q];
  }
}

// ---------------------------------------------------------------------------
// plan and launch
// ---------------------------------------------------------------------------
constexpr int WT_CUS = 256;


// output channels per block / 16: the most that divides cout, up to 3 (four
// take 36 accumulators, which leaves too few registers for the operands)
static int wgrad_mr(int cout) {
  const int t = cout / 16;
  return t % 3 == 0 ? 3 : t % 2 == 0 ? 2 : 1;
}
static void wgrad_units(int cin, int units[3]) {
  const int c16 = (cin + 15) / 16;
  // a remainder of three groups goes with a fourth that is empty: one pass over the pixels, not two
  units[0] = (c16 + 1) / 4;
  units[1] = c16 % 4 == 2;
  units[2] = c16 % 4 == 1;
}
// us of a workgroup's tile and outside its tiles, measured on eight 256^2 maps: mr 3
// 1.95 / 2.2 / 3.4 us for 16 / 32 / 64 input channels, mr 2 1.55 us for 16, 2.2 for 64;
// mr 1 1.7 for 16 (widths 16) and 2.3 for 64 (widths 112): more than is taken here, in
// nearly the ratio that is, and only the ratio shares out the chunks
static double wgrad_tile_us(int mr, int G) { return 1.35 + G * (mr == 3 ? 0.5 : mr == 2 ? 0.22 : 0.1); }
constexpr double WT_FIXED_US = 8.0;

size_t wgrad_part_floats(const WgradLayer* l, int n) {
  // every block once (chunks of any size), and one more per CU of the largest
  size_t f = 0;
  for (int k = 0; k < n; ++k) {
    const int mr = wgrad_mr(l[k].cout);
    int units[3];
    wgrad_units(l[k].cin, units);
    for (int c = 0; c < 3; ++c) f += (size_t)(l[k].cout / (16 * mr)) * units[c] * wgrad_block_floats(mr, 4 >> c);
  }
  return f + (size_t)WT_CUS * wgrad_block_floats(3, 4);
}

template <int MR>
static void wgrad_launch(WgradBatch& b, hipStream_t s) {
  // the shortest time per workgroup for which there are at most as many as CUs
  double total = 0.0;
  bool far = false;
  for (int k = 0; k < b.n; ++k) {
    WgradLayer& a = b.l[k];
    a.mt = a.cout / (16 * MR);
    wgrad_units(a.cin, a.units);
    const double nt = (double)a.B * ((a.H + WT_ROWS - 1) / WT_ROWS) * ((a.W + WT_COLS - 1) / WT_COLS);
    for (int c = 0; c < 3; ++c) total += nt * a.mt * a.units[c] * wgrad_tile_us(MR, 4 >> c);
    far |= 10.0 * a.W * std::max(a.xs, a.gzs) * 2.0 >= 2147000000.0;  // bytes between a tile's ends
  }
  for (double target = total / WT_CUS + WT_FIXED_US;; target *= 1.02) {
    b.wgs = 0;
    bool least = true;  // one chunk each
    size_t part = 0;
    int sums = 0;
    for (int k = 0; k < b.n; ++k) {
      WgradLayer& a = b.l[k];
      const int nt = a.B * ((a.H + WT_ROWS - 1) / WT_ROWS) * ((a.W + WT_COLS - 1) / WT_COLS);
      a.first = b.wgs;
      a.part = part;
      a.sum_first = sums;
      for (int c = 0; c < 3; ++c) {
        const int most = std::max(1, (int)((target - WT_FIXED_US) / wgrad_tile_us(MR, 4 >> c)));  // tiles per chunk
        a.nch[c] = (nt + most - 1) / most;
        least &= a.nch[c] == 1;
        b.wgs += a.mt * a.units[c] * a.nch[c];
        part += (size_t)a.mt * a.units[c] * a.nch[c] * wgrad_block_floats(MR, 4 >> c);
        sums += a.mt * a.units[c] * wgrad_sum_blocks(MR, 4 >> c);
      }
    }
    b.sums = sums;
    if (b.wgs <= WT_CUS || least) break;
  }
  if (far) hipLaunchKernelGGL((k_wgrad<MR, true>), dim3(b.wgs), dim3(512), 0, s, b);
  else hipLaunchKernelGGL((k_wgrad<MR, false>), dim3(b.wgs), dim3(512), 0, s, b);
  hipLaunchKernelGGL(k_wgrad_sum<MR>, dim3(b.sums), dim3(256), 0, s, b);
}

void wgrad(const WgradLayer* l, int n, float* part, hipStream_t s) {
  for (int mr = 3; mr >= 1; --mr) {
    WgradBatch b;
    b.n = 0;
    b.part = part;
    for (int k = 0; k < n; ++k)
      if (wgrad_mr(l[k].cout) == mr) b.l[b.n++] = l[k];
    if (!b.n) continue;
    switch (mr) {
      case 3: wgrad_launch<3>(b, s); break;
      case 2: wgrad_launch<2>(b, s); break;
      case 1: wgrad_launch<1>(b, s); break;
    }
  }
}

}  // namespace dn
}  // namespace kp
