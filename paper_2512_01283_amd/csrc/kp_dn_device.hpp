// kp_dn_device.hpp -- device helpers shared by the denoiser's kernels
// (kp_conv.hip, kp_denoiser.hip): BF16 conversions, 16-byte accesses, MFMA.
//
// MFMA 16x16x32 BF16 operand layout (wave64, lane l, i = l % 16, g = l / 16):
// A[i][8g + j] and B[8g + j][i] for j = 0..7 come from lane l; the result
// D[4g + j][i], j = 0..3, lands in lane l.
//
// LDS access rule of gfx950 used by the layouts below (measured with the
// SQ_LDS_BANK_CONFLICT counter on access patterns of known shape): 64 banks
// of 4 bytes; a 16-byte access is served in four passes of 16 lanes, the
// pass of lane L being (bit 5 of L, parity of bits 2, 3 and 4 of L); an
// 8-byte access in two passes of 32 consecutive lanes.  A pass without two
// lanes on one bank (at different addresses) takes one cycle.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

namespace kp {
namespace dn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest even (inputs are finite)
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ bool bf_pos(uint16_t b) { return !(b & 0x8000u) && b != 0; }

__device__ __forceinline__ u32x4 ld16(const uint16_t* p) { return *(const u32x4*)p; }
__device__ __forceinline__ void st16(uint16_t* p, u32x4 v) { *(u32x4*)p = v; }

// unpack / pack 8 BF16 held in a 16-byte vector
__device__ __forceinline__ void unpack8(u32x4 v, float* f) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    f[2 * j] = __uint_as_float(v[j] << 16);
    f[2 * j + 1] = __uint_as_float(v[j] & 0xFFFF0000u);
  }
}
__device__ __forceinline__ u32x4 pack8(const float* f) {
  u32x4 v;
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = (uint32_t)f2bf(f[2 * j]) | ((uint32_t)f2bf(f[2 * j + 1]) << 16);
  return v;
}

// two BF16 in a word, rounded to nearest even by v_cvt_pk_bf16_f32 (f2bf's results for all but NaN)
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t f2bf2(float x, float y) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2));
}

__device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                 0, 0, 0);
}

// compile-time loop: the body sees its index as a constant
template <class F, int... I>
__device__ __forceinline__ void ct_seq(F f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void ct_for(F f) {
  ct_seq(f, std::make_integer_sequence<int, N>{});
}
#define CT_INLINE __attribute__((always_inline))

}  // namespace dn
}  // namespace kp
