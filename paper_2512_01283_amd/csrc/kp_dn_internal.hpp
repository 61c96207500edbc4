// kp_dn_internal.hpp -- launch interface between the denoiser's host code
// (kp_dn_api.cpp) and its kernels (kp_denoiser.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace kp {
namespace dn {

enum { CONV_RELU = 0, CONV_PLAIN = 1, CONV_MASK = 2 };

// pixel count from which convolutions use the LDS-tiled kernel
constexpr size_t CONV_TILED_MIN_PIXELS = 1024;
inline bool conv_tiled(size_t P) { return P >= CONV_TILED_MIN_PIXELS; }

// y[p][n] (stride ys) from x[p][c] (stride xs, cin channels per tap, cin % 8 == 0)
// and GEMM weights w[nout][kp] (kp % 32 == 0, kp >= 9 cin, nout % 16 == 0).
struct ConvArgs {
  const uint16_t* x;
  int xs, cin;
  const uint16_t* w;
  int kp, nout;
  const float* bias;     // CONV_RELU
  uint16_t* y;
  int ys;
  const uint16_t* mask;  // CONV_MASK: zero the output where mask[p][n] <= 0
  int ms;
  int B, H, W;
  // only where conv_tiled(B H W):
  const uint16_t* xl;  // if set, channels 0..cl-1 (cl % 32 == 0) come from this map at half
  int xls, cl;         // resolution (stride xls), each pixel standing for a 2x2 block; x holds the rest
  uint16_t* yp;        // CONV_RELU: if set, the 2x2 means of y at half resolution (stride yps; H, W even)
  int yps;
};

// One layer's weight and bias gradients, or those of a channel range of its
// input: gw[co][kk][c] (rows of gws floats per tap, c < cin_true) and gb[co]
// += the gradients from gz[p][co] (stride gzs), the gradient of the layer's
// pre-activation output, and its input x[p][c] (stride xs, cin channels,
// cin % 8 == 0, cout % 16 == 0).
struct WgradLayer {
  const uint16_t* gz;
  int gzs, cout;
  const uint16_t* x;
  int xs, cin, cin_true, gws;
  int low;    // x lies at half resolution, each pixel standing for a 2x2 block (H, W even)
  float* gw;
  float* gb;  // null: another range's job
  int B, H, W;
  // set by the launcher: blocks of output channels; blocks of 64, 32 and 16
  // input channels and their pixel chunks; first workgroup, first block of
  // sums, first float of scratch
  int mt, units[3], nch[3], first, sum_first;
  size_t part;
};
constexpr int WGRAD_MAX = 27;  // 22 layers of a 6-level network, 5 of them in two ranges
struct WgradBatch {
  WgradLayer l[WGRAD_MAX];
  int n, wgs, sums;
  float* part;
};
// floats of a partial block: 16 mr x 9 x 16 g weights, 16 mr biases
__host__ __device__ constexpr size_t wgrad_block_floats(int mr, int g) { return (size_t)16 * mr * (9 * 16 * g + 1); }
// scratch for these layers (cin, cout) at any image size
size_t wgrad_part_floats(const WgradLayer* l, int n);
// the gradients of n <= WGRAD_MAX layers
void wgrad(const WgradLayer* l, int n, float* part, hipStream_t s);

void conv3(const ConvArgs& a, int mode, hipStream_t s);
void pool(const uint16_t* x, int xs, uint16_t* y, int ys, int B, int H, int W, int C, hipStream_t s);
void up(const uint16_t* x, int xs, uint16_t* y, int ys, int B, int H, int W, int C, hipStream_t s);
void up_bwd(const uint16_t* gy, int gys, uint16_t* gx, int gxs, const uint16_t* mask, int ms, int B, int H, int W,
            int C, hipStream_t s);
void pool_bwd_add(const uint16_t* a, int as, const uint16_t* g, int gs, const uint16_t* mask, int ms, uint16_t* dst,
                  int ds, int B, int H, int W, int C, hipStream_t s);
void sums(const double* maps, int B, int HW, int runs, double* sum, hipStream_t s);
void prep(const double* maps, const double* target, const double* sum, const int32_t* aug, int B, int H, int W,
          int runs, uint16_t* x, float* xq, float* ihat, float* tgt, hipStream_t s);
void turn(const uint16_t* x, int B, int H, int W, int code, uint16_t* y, hipStream_t s);
// code >= 0: of images transformed by it, accumulated in the original pixel order (set if first)
void head(const uint16_t* d, int C, const float* hw, const float* hb, const float* xq, float* out, int B, int H, int W,
          int code, bool first, hipStream_t s);
void loss(const float* out, const float* tgt, const float* ihat, const double* sum, int B, int HW, float* go,
          double* l, hipStream_t s);
void head_bwd(const float* go, const uint16_t* d, int C, const float* hw, float* ghw, float* ghb, uint16_t* gd,
              size_t P, hipStream_t s);
void output(const double* maps, const float* out, int B, int HW, int runs, double scale, double* dst,
            hipStream_t s);
void adam(float* p, const float* g, float* m, float* v, size_t n, float lr, int t, hipStream_t s);
void pack(const float* wf, int cout, int cin, int cin_true, int kp, int kpd, uint16_t* w, uint16_t* wd,
          hipStream_t s);
void zero(void* p, size_t bytes, hipStream_t s);

}  // namespace dn
}  // namespace kp
