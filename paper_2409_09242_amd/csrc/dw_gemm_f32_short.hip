// fp32 dual products of small models: forward products (and the data gradient through the output layer) with too few
// 64 x 64 tiles to fill the chip.
//
// Same computation as dual_gemm_f32 (C = X*Y, RC = RX*Y + X*RY of Section IV-B's forward and backward passes, products in
// three bf16 pieces).  Such a product lasts as long as the chain of its own latencies, so the contraction is cut among the
// waves of a block instead of among blocks: a block owns a 32 x 32 tile, wave w of NW takes the k-steps of 32 number w, w + NW,
// ... with its operands straight from memory (the lane that multiplies a row's or column's k loads them, splits them
// and keeps the next step's loads in flight), nothing goes through LDS and no barrier is met until the waves' partial
// tiles are added in order of w and leave with the epilogue.  Against the tiles in slices over blocks with a second
// launch that adds the slices (four workers, 128 samples): 784 -> 512 14.4 + 6.0 us, 512 -> 512 14.4 + 6.0, through 10
// classes 11.7; here 13.6, 14.4 and 9.4.  What bounds it is the way of a row's 128-byte lines, one per row and step, through L1
// (k-steps of 16, half a line each: 28 us).
#include <type_traits>

#include "dw_internal.h"
#include "dw_f32_pieces.h"

namespace dw {

namespace f32s {

constexpr int kEdge = 32;

constexpr int kStep = 32;                                    // k per step: half 0 of a wave has the first 16, half 1 the others
constexpr int kLane = kStep / 2;

// a lane's 16 k of one row (X, and Y when its k is contiguous: a row's 32 k are the 128 bytes of a cache line) or column
// (k-major Y)
struct Operand {
  const float* p;                                            // k contiguous: the row; else the column at k = 0
  // WHOLE: the step has all its k (loads without conditions go out together)
  template <bool WHOLE>
  __device__ __forceinline__ void load_row(float (&v)[kLane], int k, int K) const {
#pragma unroll
    for (int q = 0; q < kLane / 4; ++q) {
      const float4 a = WHOLE || k + 4 * q < K ? *reinterpret_cast<const float4*>(p + k + 4 * q) : make_float4(0.f, 0.f, 0.f, 0.f);
      v[4 * q] = a.x; v[4 * q + 1] = a.y; v[4 * q + 2] = a.z; v[4 * q + 3] = a.w;
    }
  }
  template <bool WHOLE>
  __device__ __forceinline__ void load_column(float (&v)[kLane], int k, int K, int ld) const {
#pragma unroll
    for (int j = 0; j < kLane; ++j) v[j] = WHOLE || k + j < K ? p[(int64_t)(k + j) * ld] : 0.f;
  }
};

// HAS_V: the +-1 operand takes part (RC += X*V); FM == 1: the R-products alone (C is in memory from an earlier probe)
template <int NW, bool Y_KC, bool HAS_RX, bool HAS_V, int EPI, int FM>
__global__ __launch_bounds__(NW * 64) void short_gemm_f32(GemmArgs a) {
  constexpr bool HAS_C = FM != 1, HAS_R = HAS_RX || HAS_V;
  const int worker = nth_active_worker(a.active_mask, blockIdx.y);
  const int tiles_m = (a.M + kEdge - 1) / kEdge;
  const int row0 = (blockIdx.x % tiles_m) * kEdge, col0 = (blockIdx.x / tiles_m) * kEdge;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lhalf = lane >> 5;
  const int K = a.K, steps = (K + kStep - 1) / kStep;

  // rows and columns past the end repeat the last ones (never stored)
  const int row = row0 + l32 < a.M ? row0 + l32 : a.M - 1, col = col0 + l32 < a.N ? col0 + l32 : a.N - 1;
  const Operand X{reinterpret_cast<const float*>(a.X) + (int64_t)worker * a.x_wstride + (int64_t)row * a.ldx};
  const Operand RX{HAS_RX ? reinterpret_cast<const float*>(a.RX) + (int64_t)worker * a.x_wstride + (int64_t)row * a.ldx : nullptr};
  const Operand Y{reinterpret_cast<const float*>(a.Y) + (int64_t)worker * a.y_wstride + (Y_KC ? (int64_t)col * a.ldy : (int64_t)col)};
  const uint32_t* zb = a.zbits + (int64_t)worker * a.z_stride;

  struct Step { float x[kLane], rx[kLane], y[kLane]; uint32_t v; };
  auto load_step = [&](Step& s, int step, auto whole) {
    constexpr bool WHOLE = decltype(whole)::value;
    const int k = step * kStep + lhalf * kLane;
    X.template load_row<WHOLE>(s.x, k, K);
    if (HAS_RX) RX.template load_row<WHOLE>(s.rx, k, K);
    if (Y_KC) Y.template load_row<WHOLE>(s.y, k, K); else Y.template load_column<WHOLE>(s.y, k, K, a.ldy);
    if (HAS_V) {
      // bits of k past the end are not read: X is zero there
      uint32_t v = 0;
      if (Y_KC) {
        const int64_t o = a.z_off + (int64_t)col * a.ldy;    // groups of four bits lie in one word
#pragma unroll
        for (int q = 0; q < kLane / 4; ++q) {
          const int64_t b = o + (WHOLE || k + 4 * q < K ? k + 4 * q : K - 4);
          v |= ((zb[b >> 5] >> (b & 31)) & 0xFu) << (4 * q);
        }
      } else {
#pragma unroll
        for (int j = 0; j < kLane; ++j) {
          const int64_t b = a.z_off + (int64_t)(WHOLE || k + j < K ? k + j : K - 1) * a.ldy + col;
          v |= ((zb[b >> 5] >> (b & 31)) & 1u) << j;
        }
      }
      s.v = v;
    }
  };
  auto load = [&](Step& s, int step) {
    if ((step + 1) * kStep <= K) load_step(s, step, std::true_type{});      // (uniform)
    else load_step(s, step, std::false_type{});
  };
  const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  floatx16 acc, racc, t, tr;
  // eight of a lane's k, from number h on
  auto multiply8 = [&](const Step& s, int h, auto whole) {
    bf16x8 v;
    if (HAS_V) {
      const uint32_t b = s.v >> h;
      v = __builtin_bit_cast(bf16x8, make_uint4(sign_pair(b, b >> 1), sign_pair(b >> 2, b >> 3), sign_pair(b >> 4, b >> 5), sign_pair(b >> 6, b >> 7)));
    }
    if constexpr (decltype(whole)::value) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (HAS_C) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(s.x[h + j], s.y[h + j], acc, 0, 0, 0);
        if (HAS_RX) racc = __builtin_amdgcn_mfma_f32_32x32x2f32(s.rx[h + j], s.y[h + j], racc, 0, 0, 0);
        if (HAS_V) racc = __builtin_amdgcn_mfma_f32_32x32x2f32(s.x[h + j], (float)v[j] * (1.f / kScale), racc, 0, 0, 0);
      }
    } else {
      auto pieces = [&](const float (&f)[kLane], bf16x8 (&o)[3]) {
        uint32_t p[3][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) split_pair<false>(f[h + 2 * q], f[h + 2 * q + 1], p[0][q], p[1][q], p[2][q]);
#pragma unroll
        for (int c = 0; c < 3; ++c) o[c] = __builtin_bit_cast(bf16x8, make_uint4(p[c][0], p[c][1], p[c][2], p[c][3]));
      };
      bf16x8 x[3], y[3];
      pieces(s.x, x);
      if (HAS_C || HAS_RX) pieces(s.y, y);
      if (HAS_C) mfma6(x, y, acc, t);
      if (HAS_V) mfma3(x, v, racc, tr);
      if (HAS_RX) {
        bf16x8 rx[3];
        pieces(s.rx, rx);
        mfma6(rx, y, racc, tr);
      }
    }
  };
  auto multiply = [&](const Step& s, auto whole) { multiply8(s, 0, whole); multiply8(s, 8, whole); };
  auto contract = [&](auto whole) {
    acc = zero; racc = zero; t = zero; tr = zero;
    Step s[2];
    if (wave < steps) load(s[0], wave);
    for (int i = wave; i < steps; i += 2 * NW) {
      if (i + NW < steps) load(s[1], i + NW);
      multiply(s[0], whole);
      if (i + NW < steps) {
        if (i + 2 * NW < steps) load(s[0], i + 2 * NW);
        multiply(s[1], whole);
      }
    }
    bool finite = true;
    if constexpr (!decltype(whole)::value) {
      if (HAS_C) finite &= join_chains(acc, t);
      if (HAS_R) finite &= join_chains(racc, tr);
    }
    return !finite;
  };
  if (K < kWholeBelow || __syncthreads_or(contract(std::false_type{}))) contract(std::true_type{});    // (see dw_f32_pieces.h)

  // partial tiles: [wave][C, RC][32][32]; lane holds column l32, rows (r/4)*8 + lhalf*4 + r%4
  extern __shared__ __attribute__((aligned(16))) float part[];
  constexpr int kTile = kEdge * kEdge, kSets = (HAS_C ? 1 : 0) + (HAS_R ? 1 : 0);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int at = ((r >> 2) * 8 + lhalf * 4 + (r & 3)) * kEdge + l32;
    if (HAS_C) part[(wave * kSets) * kTile + at] = acc[r];
    if (HAS_R) part[(wave * kSets + kSets - 1) * kTile + at] = racc[r];
  }
  __syncthreads();
  const int n = col0 + l32;
  const bool n_ok = n < a.N;
  float bias = 0.f, cz = 0.f;
  if (EPI != EPI_MASK && n_ok) {
    bias = a.bias[(int64_t)worker * a.bias_wstride + n];
    const int64_t bi = a.zb_off + n;
    if (HAS_V) cz = ((zb[bi >> 5] >> (bi & 31)) & 1u) ? 1.f : -1.f;
  }
  float* C = reinterpret_cast<float*>(a.C) + (int64_t)worker * a.c_wstride;
  float* RC = reinterpret_cast<float*>(a.RC) + (int64_t)worker * a.c_wstride;
  for (int e = tid; e < kTile; e += NW * 64) {
    const int m = row0 + (e >> 5);
    if (!n_ok || m >= a.M) continue;
    float c = 0.f, rc = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      if (HAS_C) c += part[(w * kSets) * kTile + e];
      if (HAS_R) rc += part[(w * kSets + kSets - 1) * kTile + e];
    }
    const int64_t o = (int64_t)m * a.ldc + n;
    if (EPI == EPI_RELU) {
      c += bias; rc += cz;
      const bool on = (HAS_C ? c : C[o]) > 0.f;              // (a later probe: the activation is in memory)
      if (HAS_C) C[o] = on ? c : 0.f;
      if (HAS_R) RC[o] = on ? rc : 0.f;
    } else {
      const bool on = reinterpret_cast<const float*>(a.mask_src)[(int64_t)worker * a.mask_wstride + (int64_t)m * a.ld_mask + n] > 0.f;
      if (HAS_C) C[o] = on ? c : 0.f;
      if (HAS_R) RC[o] = on ? rc : 0.f;
    }
  }
}

template <int NW, bool Y_KC, bool HAS_RX, bool HAS_V, int EPI, int FM>
static hipError_t launch(const GemmArgs& a, hipStream_t s) {
  constexpr int smem = NW * ((FM != 1 ? 1 : 0) + (HAS_RX || HAS_V ? 1 : 0)) * kEdge * kEdge * (int)sizeof(float);
  auto kern = short_gemm_f32<NW, Y_KC, HAS_RX, HAS_V, EPI, FM>;
  if (smem > 64 * 1024) {
    static LdsLimitOnce lim;
    const hipError_t e = lim.raise(reinterpret_cast<const void*>(kern), smem);
    if (e != hipSuccess) return e;
  }
  const unsigned tiles = (unsigned)(((a.M + kEdge - 1) / kEdge) * ((a.N + kEdge - 1) / kEdge));
  hipLaunchKernelGGL(kern, dim3(tiles, (unsigned)active_count(a.active_mask, a.k)), dim3(NW * 64), smem, s, a);
  return hipGetLastError();
}

}  // namespace f32s

// A forward product of M x N outputs and contraction K for each of k workers (the layout asks as well: such a product needs no
// slices).  Against the 64 x 64 tiles, in slices where there are few of them, as the step of models K-N-10 here / there:
//   K      up to 1152: faster or even (784-512, four workers of 128 samples: 76 / 82 us; 1036-340, five of 93: 77 / 83; 1036-256, two
//          of 128: 67 / 72; 1036-256, six of 256: 97 / 96).  Longer ones take too long block by block (4096-64, one of 64: the
//          product 50 / 18 us, the step 89 / 68; 1280-256, six of 256: 108 / 104) unless one block each is what most compute units
//          get, 40 to 64 tiles, four blocks to a tile: then up to 2048 (1280-512, four of 128: 87 / 98; 2048-512: 111 / 116; at 4096 163 / 157)
//   tiles  up to 128 of them as above; from there to 256 even at whole sizes (512-1024, three of 256: 108 / 103; 512-640, two of 512:
//          113 / 111) and still faster where the tiles hang over the edge (512-1036, five of 93: 101 / 111) and in first-order
//          steps (69 / 79); more of them fill the chip
bool gemm_f32_short_shape(int64_t M, int64_t N, int64_t K, int k) {
  const int64_t tiles = ((M + 63) / 64) * ((N + 63) / 64) * k;
  return tiles < 256 && K <= (tiles >= 40 && tiles <= 64 ? 2048 : 1152);
}

// Forward product, or data gradient through a layer of at most 32 outputs (the classes), of matrices in memory, no slices,
// whose 64 x 64 tiles over all workers would leave compute units idle.  Longer data gradients stay with the tiles: their
// k-major operand comes in 4-byte loads here (512 -> 512: 24 us against 11.7 + 6.0).  (Whichever workers are active: the
// choice must not depend on who steps.)
bool gemm_f32_short_ok(const GemmArgs& a) {
  if (a.x_view != VIEW_NONE || a.y_view != VIEW_NONE || a.ksplit > 1 || !(a.ry_bits || a.plain)) return false;
  if (a.epi == EPI_MASK ? a.K > f32s::kStep || (!a.plain && !a.RX) : a.epi != EPI_RELU) return false;
  return gemm_f32_short_shape(a.M, a.N, a.K, a.k);
}

template <int NW>
static hipError_t launch_forward(const GemmArgs& a, hipStream_t s) {
  using namespace f32s;
  const bool rx = a.RX != nullptr;
  if (a.plain) return launch<NW, true, false, false, EPI_RELU, 0>(a, s);
  if (a.r_only) return rx ? launch<NW, true, true, true, EPI_RELU, 1>(a, s) : launch<NW, true, false, true, EPI_RELU, 1>(a, s);
  return rx ? launch<NW, true, true, true, EPI_RELU, 0>(a, s) : launch<NW, true, false, true, EPI_RELU, 0>(a, s);
}

hipError_t launch_gemm_f32_short(const GemmArgs& a, hipStream_t s) {
  using namespace f32s;
  KernelScope ks(a.epi == EPI_MASK ? KC_GEMM_DGRAD : KC_GEMM_FWD, s);
  if (a.epi == EPI_MASK) {
    // one step, the first wave's; the others only help to write the tile (two waves 8.8 us, one 11.0)
    if (a.plain) return launch<2, false, false, false, EPI_MASK, 0>(a, s);
    return a.r_only ? launch<2, false, true, true, EPI_MASK, 1>(a, s) : launch<2, false, true, true, EPI_MASK, 0>(a, s);
  }
  return a.K > 2 * kStep ? launch_forward<8>(a, s) : launch_forward<2>(a, s);
}

}  // namespace dw
