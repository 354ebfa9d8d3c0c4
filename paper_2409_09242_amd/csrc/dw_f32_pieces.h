// fp32 products on the bf16 matrix cores (gfx950).  A float is the exact sum of three bf16 numbers
// (3 x 8 significant bits); of the nine products of two such sums the six that reach 2^-24 are multiplied
// (x1y1, x1y2, x2y1, x2y2, x1y3, x3y1), three with the +-1 operand, whose one piece is exact.  Six
// v_mfma_f32_32x32x16_bf16 (32 cycles each) replace eight v_mfma_f32_32x32x2_f32 (64 cycles each), 2.7 times less matrix
// time; with +-1 5.3 times less.  The products of the first pieces have a chain of accumulation of their own, the others,
// 2^-8 of them and less, another, and the two are added at the end: in one chain the instruction cuts small products off
// below the last bit of the running sum, always downwards (measured: -1e-8 to -4e-7 of the result's root mean square, which
// the sums over thousands of positions that follow add up).  Error of one product against 64 bits (2-norm, K = 64 / 1024 /
// 9216, normal operands): 5e-8 / 1.8e-7 / 5.9e-7, no bias; v_mfma_f32_32x32x2_f32 1.5e-7 / 5.7e-7 / 1.7e-6.
// An infinity has no pieces (inf - inf), and inf * (y1 + y2 + y3) would be no number either where y2 is 0 or of the other sign:
// the kernels compute a tile again on the fp32 matrix instruction when a result is no number.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dw {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t to_bf16x2(float a, float b) {        // round to nearest even, a in the low half
  const floatx2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
// the three pieces of a pair of floats, packed: the first is cut off (never overflows), the others are rounded
template <bool INF>
__device__ __forceinline__ void split_pair(float a, float b, uint32_t& p1, uint32_t& p2, uint32_t& p3) {
  const uint32_t au = __float_as_uint(a), bu = __float_as_uint(b);
  p1 = __builtin_amdgcn_perm(bu, au, 0x07060302u);
  float ra = a - __uint_as_float(au & 0xFFFF0000u), rb = b - __uint_as_float(bu & 0xFFFF0000u);
  if (INF) {                                                 // inf - inf would be a NaN
    if ((au & 0x7FFFFFFFu) == 0x7F800000u) ra = 0.f;
    if ((bu & 0x7FFFFFFFu) == 0x7F800000u) rb = 0.f;
  }
  p2 = to_bf16x2(ra, rb);
  ra -= __uint_as_float(p2 << 16); rb -= __uint_as_float(p2 & 0xFFFF0000u);
  p3 = to_bf16x2(ra, rb);
}
template <bool INF, int N>                                   // N pairs
__device__ __forceinline__ void split_pairs(const float (&x)[2 * N], uint32_t (&p)[3][N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) split_pair<INF>(x[2 * i], x[2 * i + 1], p[0][i], p[1][i], p[2][i]);
}
// +-1 as a pair of bf16 from two bits (bit set: +1)
__device__ __forceinline__ uint32_t sign_pair(uint32_t b0, uint32_t b1) {
  return 0xBF80BF80u ^ ((b0 & 1u) << 15) ^ ((b1 & 1u) << 31);
}

// the products of one k-step of 16 of two numbers in three pieces: those of the first pieces to m, the others to t
__device__ __forceinline__ void mfma6(const bf16x8 (&x)[3], const bf16x8 (&y)[3], floatx16& m, floatx16& t) {
  m = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], y[0], m, 0, 0, 0);
  t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[2], y[0], t, 0, 0, 0);
  t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], y[2], t, 0, 0, 0);
  t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[1], y[1], t, 0, 0, 0);
  t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[1], y[0], t, 0, 0, 0);
  t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], y[1], t, 0, 0, 0);
}
__device__ __forceinline__ void mfma3(const bf16x8 (&x)[3], const bf16x8& v, floatx16& m, floatx16& t) {
  m = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], v, m, 0, 0, 0);
  t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[2], v, t, 0, 0, 0);
  t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[1], v, t, 0, 0, 0);
}
}  // namespace dw
