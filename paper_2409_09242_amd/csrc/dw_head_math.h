// Softmax cross-entropy of one sample and its derivative along Rs (Section II eq.(2) with the softmax loss; the
// R-derivative is the one of Section IV-B's Hessian-vector product): by one thread, and by a group of 16 lanes that hold the
// logits already.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

#include <utility>

#include "dw.h"

namespace dw {

// s[c], rs[c]: logits and their directional derivative for c < C (entries beyond C are ignored), y: the label.
// d[c] = (p_c - [c == y]) * invB, rd[c] = p_c (Rs_c - <p, Rs>) * invB for c < C, zero beyond.  Returns -log p_y.
__device__ __forceinline__ float head_row(const float (&s_in)[DW_MAX_CLASSES], const float (&rs_in)[DW_MAX_CLASSES],
                                          int y, int C, float invB, float (&d)[DW_MAX_CLASSES],
                                          float (&rd)[DW_MAX_CLASSES]) {
  float s[DW_MAX_CLASSES], rs[DW_MAX_CLASSES];
  float mx = -INFINITY;
  int amax = 0;
#pragma unroll
  for (int c = 0; c < DW_MAX_CLASSES; ++c) {
    s[c] = c < C ? s_in[c] : -INFINITY;
    rs[c] = c < C ? rs_in[c] : 0.f;
    if (s[c] > mx) { mx = s[c]; amax = c; }
  }
  // e_c = exp(s_c - max); the largest term is exactly 1, so sums that leave it (or the label's term)
  // out keep full relative precision when the prediction is confident
  float rest_max = 0.f, rest_y = 0.f, sy = 0.f;
#pragma unroll
  for (int c = 0; c < DW_MAX_CLASSES; ++c) {
    const float e = c < C ? expf(s[c] - mx) : 0.f;
    if (c == y) sy = s[c] - mx;
    if (c != amax) rest_max += e;
    if (c != y) rest_y += e;
    s[c] = e;
  }
  const float sum = 1.0f + rest_max;
  const float inv = 1.0f / sum;
#pragma unroll
  for (int c = 0; c < DW_MAX_CLASSES; ++c) s[c] *= inv;   // p_c
  const float one_minus_py = rest_y * inv;         // 1 - p_y without cancellation
#pragma unroll
  for (int c = 0; c < DW_MAX_CLASSES; ++c) {
    d[c] = 0.f; rd[c] = 0.f;
    if (c < C) {
      d[c] = (c == y ? -one_minus_py : s[c]) * invB;  // d(mean loss)/d s_L = (p - onehot)/B
      // its derivative along Rs_L: p_c (Rs_c - <p, Rs>) / B, with Rs_c - <p, Rs> written as
      // sum_c' p_c' (Rs_c - Rs_c') so that a confident prediction does not cancel
      float ctr = 0.f;
#pragma unroll
      for (int c2 = 0; c2 < DW_MAX_CLASSES; ++c2) ctr += s[c2] * (rs[c] - rs[c2]);
      rd[c] = s[c] * ctr * invB;
    }
  }
  return log1pf(rest_max) - sy;                    // -log p_y = log(sum_c e_c) - (s_y - max)
}

// another lane of the same row of 16 lanes, without a trip through LDS.  kRowLane + n: lane n for all; kRowTurn + n: the lane n further on
constexpr int kRowLane = 0x150, kRowTurn = 0x120;
template <int CTRL>
__device__ __forceinline__ float row_move(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}
// the sum (in 64 bits: rounded once, whichever order) and the largest of a row's 16, the same bits in all its lanes
template <int CTRL>
__device__ __forceinline__ double row_move(double x) {
  const uint2 u = __builtin_bit_cast(uint2, x);
  return __builtin_bit_cast(double, make_uint2((uint32_t)__builtin_amdgcn_update_dpp(0, (int)u.x, CTRL, 0xF, 0xF, false),
                                               (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u.y, CTRL, 0xF, 0xF, false)));
}
__device__ __forceinline__ double row_sum(float f) {
  double x = (double)f;
  x += row_move<kRowTurn + 8>(x); x += row_move<kRowTurn + 4>(x); x += row_move<kRowTurn + 2>(x);
  return x + row_move<kRowTurn + 1>(x);
}
__device__ __forceinline__ float row_max(float x) {
  x = fmaxf(x, row_move<kRowTurn + 8>(x)); x = fmaxf(x, row_move<kRowTurn + 4>(x)); x = fmaxf(x, row_move<kRowTurn + 2>(x));
  return fmaxf(x, row_move<kRowTurn + 1>(x));
}
// sum over the row's lanes c of p_c (rs - rs_c)
template <int... N>
__device__ __forceinline__ float row_centred(float p, float rs, std::integer_sequence<int, N...>) {
  float ctr = 0.f;
  ((ctr = fmaf(row_move<kRowLane + N>(p), rs - row_move<kRowLane + N>(rs), ctr)), ...);
  return ctr;
}

// The same for the 16 lanes of a row that hold a sample's logits, one class each: lane n has s = s_n, rs = Rs_n and receives
// d_n and Rd_n; the loss is log1pf(rest) - sy (left to the caller: off the way to the errors).  A sample by one lane is a chain of
// some 1500 instructions, by 16 of a tenth (output layer 512 wide, 10 classes, four workers of 128 samples: kernel 11.7 -> 9.4 us).
// All 64 lanes of the wave take part.
__device__ __forceinline__ void head_lanes(float s, float rs, int n, int y, int C, float invB, float& d, float& rd, float& rest, float& sy) {
  static_assert(DW_MAX_CLASSES == 16, "a row of lanes holds a sample's logits");
  s = n < C ? s : -INFINITY;
  rs = n < C ? rs : 0.f;
  const float mx = row_max(s > -INFINITY ? s : -INFINITY);             // (a logit that is no number is not the largest)
  const uint32_t at_max = (uint32_t)(__ballot(s == mx) >> (threadIdx.x & 48)) & 0xFFFFu;
  const int amax = mx > -INFINITY ? __builtin_ctz(at_max) : 0;         // the first one
  const float e = n < C ? expf(s - mx) : 0.f;
  // sums that leave the largest term, exactly 1, or the label's out, as in head_row
  const double others = row_sum(n == amax ? 0.f : e);
  rest = (float)others;
  const float rest_y = (float)row_sum(n == y ? 0.f : e);
  sy = (float)row_sum(n == y ? s - mx : 0.f);
  const float inv = 1.0f / (float)(1.0 + others), p = e * inv;
  const float ctr = row_centred(p, rs, std::make_integer_sequence<int, DW_MAX_CLASSES>{});
  d = n < C ? (n == y ? -(rest_y * inv) : p) * invB : 0.f;
  rd = n < C ? p * ctr * invB : 0.f;
}

}  // namespace dw
