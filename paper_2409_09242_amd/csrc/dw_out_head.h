// The rows of an output-layer block (16 samples, at most 16 classes): the waves' partial products become logits and go
// through the softmax head without going to memory.  Shared by the fp32 and the bf16 output-layer kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "dw_internal.h"
#include "dw_device_util.h"
#include "dw_head_math.h"

namespace dw {

// part: [wave][S, RS][sample][class], complete; block of 256 threads.  Writes d_L, Rd_L (and their bf16 copies) and the
// block's loss into its slot of loss_part.
template <int NW>
__device__ __forceinline__ void out_head_rows(const float (&part)[NW][2][DW_MAX_CLASSES][DW_MAX_CLASSES + 1], const GemmArgs& a,
                                              const HeadArgs& h, float* loss_part, int worker, int row0, const uint32_t* zb) {
  __shared__ float row_loss[DW_MAX_CLASSES];
  const int tid = threadIdx.x;
  const int m = tid >> 4, n = tid & 15;                   // one 16-lane group per sample, one lane per class
  float s = 0.f, rs = 0.f;
  if (n < a.N) {
#pragma unroll
    for (int w = 0; w < NW; ++w) { s += part[w][0][m][n]; rs += part[w][1][m][n]; }
    const int64_t bi = a.zb_off + n;
    s += a.bias[(int64_t)worker * a.bias_wstride + n];
    rs += ((zb[bi >> 5] >> (bi & 31)) & 1u) ? 1.f : -1.f;
  }
  const int row = row0 + m;
  const int yrow = row < a.M ? row : a.M - 1;
  const int y = h.y[(int64_t)worker * h.B + yrow];
  float dn, rdn, rest, sy;
  head_lanes(s, rs, n, y, h.C, 1.0f / (float)h.B, dn, rdn, rest, sy);
  if (row < a.M && n < h.ld) {
    const int64_t o = ((int64_t)worker * h.B + row) * h.ld + n;
    h.delta[o] = dn;
    h.Rdelta[o] = rdn;
    if (h.delta_b16) { h.delta_b16[o] = f32_to_bf16_rne(dn); h.Rdelta_b16[o] = f32_to_bf16_rne(rdn); }
  }
  if (n == 0) row_loss[m] = row < a.M ? log1pf(rest) - sy : 0.f;
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;                                       // (16 sums in fp32 would be off by a last bit or two)
#pragma unroll
    for (int r = 0; r < DW_MAX_CLASSES; ++r) t += (double)row_loss[r];
    loss_part[(int64_t)worker * gridDim.x + blockIdx.x] = (float)t;
  }
}

}  // namespace dw
