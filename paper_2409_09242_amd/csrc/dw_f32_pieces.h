// fp32 products on the bf16 matrix cores (gfx950), by a published method (G. Henry, P. T. P. Tang, A. Heinecke, "Leveraging the
// bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", ARITH 2019).  A float is the exact sum of three
// bf16 numbers (3 x 8 significant bits), each the rounding of what the ones before leave: for x in [1, 2) the second is at most
// 2^-8 and the third 2^-17.  Of the nine products of two such sums six are multiplied (x1y1, x1y2, x2y1, x2y2, x1y3, x3y1),
// three with the +-1 operand, whose one piece is exact; the others, x2y3 and x3y2, are at most 2^-25 each (2^-23 with a first piece
// that is cut off instead of rounded).  Six v_mfma_f32_32x32x16_bf16 (32 cycles each) replace eight v_mfma_f32_32x32x2_f32 (64
// cycles each), 2.7 times less matrix time; with +-1 5.3 times less.  The products of the first pieces have a chain of
// accumulation of their own, the others, 2^-8 of them and less, another, and the two are added at the end: in one chain the
// instruction cuts small products off below the last bit of the running sum, always downwards (measured: -1e-8 to -4e-7 of the
// result's root mean square, which the sums over thousands of positions that follow add up).
//
// Error of one product against 64 bits, normal operands, 2-norm of all / largest over sum |x||y|, no bias (in brackets
// v_mfma_f32_32x32x2_f32):
//   K = 1   2.6e-8 / 9.0e-8 (2.5e-8 / 5.9e-8)      K = 4   2.7e-8 / 1.3e-7 (4.0e-8 / 1.5e-7)     K = 128   6.4e-8 (2.1e-7)
//   K = 2   2.6e-8 / 1.2e-7 (3.1e-8 / 1.1e-7)      K = 16  3.2e-8 / 1.1e-7 (7.3e-8 / 2.1e-7)     K = 512   1.3e-7 (4.0e-7)
//   K = 3   2.7e-8 / 1.2e-7 (3.6e-8 / 1.3e-7)      K = 32  3.9e-8 / 1.1e-7 (1.0e-7 / 2.4e-7)     K = 2048  2.7e-7 (8.1e-7)
// A contraction of one or two is closer on the fp32 instruction and goes there (kWholeBelow; it lasts no longer at such sizes).
//
// The pieces are those of 2^24 times the number, so that every piece of every fp32 number, the subnormal ones among them, is a
// normal bf16 number (the matrix cores lose subnormal ones: operands of 2^-118 and 32 k, 2^24-fold pieces 3.9e-8, pieces of the
// number itself 8.8e-6, of 2^-130 3.6e-2); the +-1 operand is +-2^24 likewise, the results are 2^48-fold and leave through
// kUnscale.  That takes one multiplication per element (3072-1024^3, eight workers: 935 -> 959 us a step) and leaves operands
// below 2^104 and results below 2^80.
//
// A larger operand or result, an infinity (which has no pieces: inf - inf) or a NaN gives a result that is infinite or no number:
// the kernels then compute the tile again from the whole floats on the fp32 matrix instruction, which gives what such operands give.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dw {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t to_bf16x2(float a, float b) {        // round to nearest even, a in the low half
  const floatx2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
constexpr float kScale = 0x1p24f, kUnscale = 0x1p-48f;
constexpr int kWholeBelow = 3;             // contractions shorter than this run on the fp32 instruction
// the three pieces of a pair of floats, packed.  HALVES: the two halves of the floats' own bits instead, for the pass on the fp32
// instruction
template <bool HALVES>
__device__ __forceinline__ void split_pair(float a, float b, uint32_t& p1, uint32_t& p2, uint32_t& p3) {
  if (HALVES) {
    const uint32_t au = __float_as_uint(a), bu = __float_as_uint(b);
    p1 = __builtin_amdgcn_perm(bu, au, 0x07060302u);
    p2 = __builtin_amdgcn_perm(bu, au, 0x05040100u);
    p3 = 0u;
    return;
  }
  a *= kScale; b *= kScale;
  p1 = to_bf16x2(a, b);
  float ra = a - __uint_as_float(p1 << 16), rb = b - __uint_as_float(p1 & 0xFFFF0000u);
  p2 = to_bf16x2(ra, rb);
  ra -= __uint_as_float(p2 << 16); rb -= __uint_as_float(p2 & 0xFFFF0000u);
  p3 = to_bf16x2(ra, rb);
}
template <bool HALVES, int N>                                // N pairs
__device__ __forceinline__ void split_pairs(const float (&x)[2 * N], uint32_t (&p)[3][N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) split_pair<HALVES>(x[2 * i], x[2 * i + 1], p[0][i], p[1][i], p[2][i]);
}
// +-2^24 as a pair of bf16 from two bits (bit set: +)
__device__ __forceinline__ uint32_t sign_pair(uint32_t b0, uint32_t b1) {
  return 0xCB80CB80u ^ ((b0 & 1u) << 15) ^ ((b1 & 1u) << 31);
}
// the two chains of a result (below) put together: the result, and whether it is finite
__device__ __forceinline__ bool join_chains(floatx16& m, const floatx16& t) {
  m += t;
  bool finite = true;
#pragma unroll
  for (int r = 0; r < 16; ++r) finite &= __builtin_fabsf(m[r]) < __builtin_inff();
  m *= kUnscale;
  return finite;
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
