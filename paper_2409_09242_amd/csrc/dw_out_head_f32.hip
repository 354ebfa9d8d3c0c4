// fp32 output layer and softmax head in one kernel.
//
// S = A W^T + b and RS = RA W^T + A V^T + c (Section IV-B) with W [C][K], C <= 16 classes, followed at once by the
// softmax cross-entropy of the rows and its R-derivative (dw_head_math.h): the logits never go to memory.  For the
// small models this replaces three short launches in a row (a product with a handful of tiles, the sum of its slices,
// the head) by one.  A block owns 16 samples; its four waves take a quarter of the contraction each with the
// 16 x 16 x 4 MFMA, every lane loading 16 bytes (4 consecutive k) of A, RA and W per step, and the four partial tiles
// are added in wave order through LDS.  A 16-lane group then holds one sample's 16 logits, a class each, and runs the head
// on them together (head_lanes).  The loss of the block's samples goes to one slot per (worker, block);
// the update's kernel adds a worker's slots when the caller wants the loss.
//
// Few samples and a long contraction leave a handful of blocks walking all of it.  There the contraction is cut into slices
// over the grid, whose partial logits go to scratch, and a second launch adds them in order and runs the head
// (out_head_f32_slices).
#include "dw_out_head.h"

namespace dw {

typedef float f32o_x4 __attribute__((ext_vector_type(4)));

namespace f32o {

constexpr int ROWS = 16, NT = 256, NW = NT / 64, KSTEP = 16;
static_assert(DW_MAX_CLASSES == ROWS, "a 16-lane group holds one sample's logits, one class per lane");

// grid: (ceil(M / 16), active workers, slices of the contraction); requirements in out_head_f32_ok.  SLICED: partial logits to
// slices[slice][worker][block][S, RS][sample][class]
template <bool SLICED>
__global__ __launch_bounds__(NT) void out_head_f32_kernel(GemmArgs a, HeadArgs h, float* loss_part, float* slices) {
  const int worker = nth_active_worker(a.active_mask, blockIdx.y);
  const int row0 = blockIdx.x * ROWS;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kg = lane >> 4;               // operand row (A) or column (W), and which 4 of the 16 k
  // the slice (whole groups of 64 but for the last one's end) and this wave's share of it
  const int klen = SLICED ? ((a.K + gridDim.z - 1) / gridDim.z + NW * KSTEP - 1) / (NW * KSTEP) * (NW * KSTEP) : a.K;
  const int k0s = SLICED ? ((int)blockIdx.z * klen < a.K ? (int)blockIdx.z * klen : a.K) : 0;    // (rounding up may leave none for the last)
  const int k1s = SLICED && k0s + klen < a.K ? k0s + klen : a.K;
  const int kspan = (k1s - k0s + NW * KSTEP - 1) / (NW * KSTEP) * KSTEP;
  const int kbeg = k0s + wave * kspan, kend = kbeg + kspan < k1s ? kbeg + kspan : k1s;
  const int arow = row0 + r16 < a.M ? row0 + r16 : a.M - 1;   // rows past the end repeat the last one (never stored)

  const float* X = reinterpret_cast<const float*>(a.X) + (int64_t)worker * a.x_wstride + (int64_t)arow * a.ldx;
  const bool has_rx = a.RX != nullptr;
  const float* RX = has_rx ? reinterpret_cast<const float*>(a.RX) + (int64_t)worker * a.x_wstride + (int64_t)arow * a.ldx
                           : X;
  const bool col_ok = r16 < a.N;
  const int wrow = col_ok ? r16 : 0;                       // lanes of padding columns read row 0 and multiply by zero
  const float* W = reinterpret_cast<const float*>(a.Y) + (int64_t)worker * a.y_wstride + (int64_t)wrow * a.ldy;
  const uint32_t* zb = a.zbits + (int64_t)worker * a.z_stride;
  const int64_t zbit0 = a.z_off + (int64_t)wrow * a.ldy;    // multiple of 4: the 4 bits sit in one word

  f32o_x4 acc = {0.f, 0.f, 0.f, 0.f}, racc = {0.f, 0.f, 0.f, 0.f};

  const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
  if ((k1s - k0s) % (NW * KSTEP) == 0) {                   // (512 wide: 12 us, the form below 15)
    for (int k0 = kbeg; k0 < kbeg + kspan; k0 += KSTEP) {
      const float4 x4 = *reinterpret_cast<const float4*>(X + k0 + kg * 4);
      const float4 rx4 = has_rx ? *reinterpret_cast<const float4*>(RX + k0 + kg * 4) : make_float4(0.f, 0.f, 0.f, 0.f);
      const float4 w4 = col_ok ? *reinterpret_cast<const float4*>(W + k0 + kg * 4) : make_float4(0.f, 0.f, 0.f, 0.f);
      const int64_t bi = zbit0 + k0 + kg * 4;
      const uint32_t bits = col_ok ? (zb[bi >> 5] >> (bi & 31)) & 0xFu : 0u;
      const float x[4] = {x4.x, x4.y, x4.z, x4.w}, rx[4] = {rx4.x, rx4.y, rx4.z, rx4.w}, w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float v = col_ok ? (((bits >> j) & 1u) ? 1.f : -1.f) : 0.f;
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j], w[j], acc, 0, 0, 0);
        racc = __builtin_amdgcn_mfma_f32_16x16x4f32(rx[j], w[j], racc, 0, 0, 0);
        racc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j], v, racc, 0, 0, 0);
      }
    }
  } else {
    // four steps' loads go out together
    constexpr int BATCH = 4;
    for (int kb = kbeg; kb < kend; kb += BATCH * KSTEP) {
      float4 x4[BATCH], rx4[BATCH], w4[BATCH];
      uint32_t bits[BATCH];
      bool live[BATCH];
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        // past the end (the last steps may be short or missing; K is a multiple of 4): the last four k again, times zero
        const int k = kb + u * KSTEP + kg * 4, kc = k < kend ? k : a.K - 4;
        x4[u] = *reinterpret_cast<const float4*>(X + kc);
        rx4[u] = has_rx ? *reinterpret_cast<const float4*>(RX + kc) : zero4;
        w4[u] = *reinterpret_cast<const float4*>(W + kc);
        const int64_t bi = zbit0 + kc;
        bits[u] = zb[bi >> 5] >> (bi & 31);
        live[u] = k < kend;
      }
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const float xs[4] = {x4[u].x, x4[u].y, x4[u].z, x4[u].w}, rxs[4] = {rx4[u].x, rx4[u].y, rx4[u].z, rx4[u].w};
        const float ws[4] = {w4[u].x, w4[u].y, w4[u].z, w4[u].w};
        float x[4], rx[4], w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) { x[j] = live[u] ? xs[j] : 0.f; rx[j] = live[u] ? rxs[j] : 0.f; w[j] = live[u] && col_ok ? ws[j] : 0.f; }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float v = col_ok ? (((bits[u] >> j) & 1u) ? 1.f : -1.f) : 0.f;
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j], w[j], acc, 0, 0, 0);
          racc = __builtin_amdgcn_mfma_f32_16x16x4f32(rx[j], w[j], racc, 0, 0, 0);
          racc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j], v, racc, 0, 0, 0);
        }
      }
    }
  }

  // partial tiles of the four waves: element (row, col) of a wave sits in lane col + 16*(row/4), register row%4
  __shared__ float part[NW][2][ROWS][ROWS + 1];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    part[wave][0][kg * 4 + r][r16] = acc[r];
    part[wave][1][kg * 4 + r][r16] = racc[r];
  }
  __syncthreads();
  if (SLICED) {
    const int m = tid >> 4, n = tid & 15;
    float s = 0.f, rs = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) { s += part[w][0][m][n]; rs += part[w][1][m][n]; }
    float* out = slices + (((int64_t)blockIdx.z * a.k + worker) * gridDim.x + blockIdx.x) * (2 * NT);
    out[tid] = s;
    out[NT + tid] = rs;
  } else {
    out_head_rows<NW>(part, a, h, loss_part, worker, row0, zb);
  }
}

// the slices of a block's logits in order, then the head
__global__ __launch_bounds__(NT) void out_head_slices_kernel(GemmArgs a, HeadArgs h, float* loss_part, const float* slices, int n_slices) {
  const int worker = nth_active_worker(a.active_mask, blockIdx.y);
  const int tid = threadIdx.x;
  __shared__ float part[1][2][ROWS][ROWS + 1];
  const float* in = slices + ((int64_t)worker * gridDim.x + blockIdx.x) * (2 * NT) + tid;
  const int64_t step = (int64_t)a.k * gridDim.x * (2 * NT);
  float s = 0.f, rs = 0.f;
#pragma unroll 8
  for (int i = 0; i < n_slices; ++i) { s += in[i * step]; rs += in[i * step + NT]; }
  part[0][0][tid >> 4][tid & 15] = s;
  part[0][1][tid >> 4][tid & 15] = rs;
  __syncthreads();
  out_head_rows<1>(part, a, h, loss_part, worker, blockIdx.x * ROWS, a.zbits + (int64_t)worker * a.z_stride);
}

}  // namespace f32o

// Slices of an output layer's contraction K for k workers of M samples: enough for 512 blocks, each at least 512 long; 1: none.
// Measured without hidden layers, whole and cut: 64 samples, one worker: 2048 wide 26 and 15 us, 8196 wide 81 and 17 (512 wide 13
// whole); 256 blocks in two slices each: 2048 wide 27 and 24 us, 8196 wide 82 and 59.  More blocks than that are not cut.
int out_head_f32_slices(int64_t M, int64_t K, int k) {
  const int64_t blocks = (M + f32o::ROWS - 1) / f32o::ROWS * k;
  if (K < 2048 || blocks > 256) return 1;
  const int64_t fill = 512 / blocks, most = K / 512;
  return (int)(fill < most ? fill : most);
}
size_t out_head_f32_slice_bytes(int64_t M, int64_t K, int k) {
  const int s = out_head_f32_slices(M, K, k);
  return s > 1 ? (size_t)s * k * ((M + f32o::ROWS - 1) / f32o::ROWS) * (2 * f32o::NT) * sizeof(float) : 0;
}

// the fp32 output layer's forward product (linear epilogue, at most 16 columns) with operands that 16-byte loads can
// address and sign bits that come four to a word
bool out_head_f32_ok(const GemmArgs& a) {
  if (a.epi != EPI_LINEAR || !(a.ry_bits || a.plain) || !a.x_kcontig || !a.y_kcontig || a.ksplit > 1) return false;
  if (a.N < 1 || a.N > f32o::ROWS || a.M < 1) return false;
  if (a.K < 1 || a.K % 4 != 0) return false;
  if (a.ldx % 4 != 0 || a.ldy % 4 != 0 || a.x_wstride % 4 != 0 || a.y_wstride % 4 != 0 || a.z_off % 4 != 0) return false;
  if ((reinterpret_cast<uintptr_t>(a.X) & 15u) || (reinterpret_cast<uintptr_t>(a.Y) & 15u) ||
      (a.RX && (reinterpret_cast<uintptr_t>(a.RX) & 15u)))
    return false;
  return true;
}

// loss_part: at least k * ceil(M / 16) floats; slices: scratch of
// out_head_f32_slice_bytes
hipError_t launch_out_head_f32(const GemmArgs& a, const HeadArgs& h, float* loss_part, float* slices, hipStream_t s) {
  KernelScope ks(KC_HEAD, s);
  const int n_slots = (a.M + f32o::ROWS - 1) / f32o::ROWS;
  const dim3 grid((unsigned)n_slots, (unsigned)active_count(a.active_mask, a.k));
  const int n_slices = out_head_f32_slices(a.M, a.K, a.k);
  if (n_slices > 1) {
    hipLaunchKernelGGL(f32o::out_head_f32_kernel<true>, dim3(grid.x, grid.y, (unsigned)n_slices), dim3(f32o::NT), 0, s, a, h, loss_part, slices);
    hipLaunchKernelGGL(f32o::out_head_slices_kernel, grid, dim3(f32o::NT), 0, s, a, h, loss_part, slices, n_slices);
  } else {
    hipLaunchKernelGGL(f32o::out_head_f32_kernel<false>, grid, dim3(f32o::NT), 0, s, a, h, loss_part, slices);
  }
  return hipGetLastError();
}

}  // namespace dw
