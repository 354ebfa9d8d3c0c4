// fp32 dual products of small models: forward products and data gradients with too few 64 x 64 tiles to fill the chip.
//
// Same computation as dual_gemm_f32 (C = X*Y, RC = RX*Y + X*RY of Section IV-B's forward and backward passes, products in
// three bf16 pieces).  Such a product lasts as long as the chain of its own latencies, so the contraction is cut among the
// waves of a block instead of among blocks: a block owns a 32 x 32 tile, wave w of NW takes the k-steps of 32 number w, w + NW,
// ..., and no barrier is met until the waves' partial tiles are added in order of w and leave with the epilogue.  A wave loads
// whole 128-byte lines, eight lanes each (two steps in flight), and turns them in a region of LDS of its own so that a lane gets
// the 16 k of the row it multiplies; k-major operands (W in the data gradient) come as 32 columns of 32 k and are read by columns.
// Four workers, 128 samples: forward 784 -> 512 14.1 us, 512 -> 512 12.6 (each lane loading its own row, a line per lane and step:
// 14.9 both), data gradient 512 -> 512 12.3 (64 x 64 tiles in slices and a launch that adds them 13.3 + 5.5), first-order 7.9 (8.7 + 4.8).
// Where 12.6 us go, by clock readings in a block of eight waves: until the first loads are out 1.1 us, until they are all there 3,
// the two steps of each wave 4.5 (splitting and multiplying by turns, two waves to a SIMD), joining the partial tiles 1.2, the rest
// is launch and drain.  Loads arrive at 24 bytes a clock and compute unit, a third of what L1 passes on when it hits.
#include <type_traits>

#include "dw_internal.h"
#include "dw_f32_pieces.h"

namespace dw {

namespace f32s {

constexpr int kEdge = 32;
constexpr int kStep = 32;                                    // k per step: half 0 of a wave has the first 16, half 1 the others
constexpr int kLane = kStep / 2;

// 32 x 32 floats of an operand on their way through a wave's LDS.  In memory and in LDS lines of 32 floats: a row's 32 k (k
// contiguous), or 32 columns of one k.
// Rows: 16-byte unit u of row r sits at place u ^ (r & 7), so that eight rows' units of the same number use different banks.
constexpr int kRowsFloats = kEdge * kStep;
__device__ __forceinline__ int row_unit(int row, int unit) { return row * kStep + ((unit ^ (row & 7)) << 2); }
// Columns: the second half's 16 k start 32 banks further on, so that the two halves of a wave read different banks
constexpr int kColumnsFloats = kEdge * kStep + kEdge;
__device__ __forceinline__ int column_line(int k) { return k * kEdge + (k >= kLane ? kEdge : 0); }

constexpr int wave_floats(bool y_kc, bool has_rx, bool has_v) {
  return kRowsFloats * (has_rx ? 2 : 1) + (y_kc ? kRowsFloats : kColumnsFloats + (has_v ? kStep : 0));
}

// what a wave has written to its region is there for its reads
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// HAS_V: the +-1 operand takes part (RC += X*V); FM == 1: the R-products alone (C is in memory from an earlier probe)
template <int NW, bool Y_KC, bool HAS_RX, bool HAS_V, int EPI, int FM>
__global__ __launch_bounds__(NW * 64) void short_gemm_f32(GemmArgs a) {
  constexpr bool HAS_C = FM != 1, HAS_R = HAS_RX || HAS_V;
  const unsigned tiles_m = (a.M + kEdge - 1) / kEdge, tiles = tiles_m * ((a.N + kEdge - 1) / kEdge), logical = xcd_unit();
  const unsigned slot = logical / tiles, tile = logical - slot * tiles;
  if (slot >= (unsigned)active_count(a.active_mask, a.k)) return;
  const int worker = nth_active_worker(a.active_mask, slot);
  const int row0 = (tile % tiles_m) * kEdge, col0 = (tile / tiles_m) * kEdge;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lhalf = lane >> 5;
  const int line = lane >> 3, unit = lane & 7;               // loads: line 8 i + `line` of 32, 16-byte unit of the line
  const int K = a.K, steps = (K + kStep - 1) / kStep;

  extern __shared__ __attribute__((aligned(16))) float lds[];
  float* Xl = lds + wave * wave_floats(Y_KC, HAS_RX, HAS_V);
  float* RXl = Xl + kRowsFloats;
  float* Yl = Xl + kRowsFloats * (HAS_RX ? 2 : 1);
  uint32_t* Vl = reinterpret_cast<uint32_t*>(Yl + kColumnsFloats);

  // rows and columns past the end repeat the last ones (never stored); operands of a worker have fewer than 2^31 elements
  const float* X = reinterpret_cast<const float*>(a.X) + (int64_t)worker * a.x_wstride;
  const float* RX = HAS_RX ? reinterpret_cast<const float*>(a.RX) + (int64_t)worker * a.x_wstride : nullptr;
  const float* Y = reinterpret_cast<const float*>(a.Y) + (int64_t)worker * a.y_wstride;
  const uint32_t* zb = a.zbits + (int64_t)worker * a.z_stride;
  int xo[4], yo[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = row0 + 8 * i + line, c = col0 + 8 * i + line;
    xo[i] = (r < a.M ? r : a.M - 1) * a.ldx + unit * 4;
    yo[i] = (c < a.N ? c : a.N - 1) * a.ldy + unit * 4;
  }
  const int ycol = col0 + unit * 4 < a.N ? col0 + unit * 4 : a.N - 4;           // k-major: this lane's four columns (N is a multiple of 4)
  const int col = col0 + l32 < a.N ? col0 + l32 : a.N - 1;

  struct Step { float4 x[4], rx[4], y[4]; uint32_t v0, v1; int sh; };
  auto load_step = [&](Step& s, int k0, auto whole) {
    constexpr bool WHOLE = decltype(whole)::value;
    const bool ok = WHOLE || k0 + unit * 4 < K;              // (rows end at a multiple of 4: the widths are, and the output layer's errors have zeros from the last class to 16)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s.x[i] = ok ? *reinterpret_cast<const float4*>(X + xo[i] + k0) : make_float4(0.f, 0.f, 0.f, 0.f);
      if (HAS_RX) s.rx[i] = ok ? *reinterpret_cast<const float4*>(RX + xo[i] + k0) : make_float4(0.f, 0.f, 0.f, 0.f);
      if (Y_KC) {
        s.y[i] = ok ? *reinterpret_cast<const float4*>(Y + yo[i] + k0) : make_float4(0.f, 0.f, 0.f, 0.f);
      } else {
        const int k = k0 + 8 * i + line;
        s.y[i] = WHOLE || k < K ? *reinterpret_cast<const float4*>(Y + (int64_t)k * a.ldy + ycol) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
    if (HAS_V) {
      // the words that hold a lane's signs: 16 of its row (k contiguous), or 32 of line `l32` (the bits after the last are not
      // read; X is zero for k past the end)
      int64_t first, last;
      if (Y_KC) {
        const int k = k0 + lhalf * kLane, kf = WHOLE || k < K ? k : K - 4;
        first = a.z_off + (int64_t)col * a.ldy + kf;
        last = first + (WHOLE || kf + kLane <= K ? kLane : K - kf) - 1;
      } else {
        const int k = WHOLE || k0 + l32 < K ? k0 + l32 : K - 1;
        first = a.z_off + (int64_t)k * a.ldy + col0;
        last = first + (col0 + kEdge <= a.N ? kEdge : a.N - col0) - 1;
      }
      s.v0 = zb[first >> 5]; s.v1 = zb[last >> 5];
      s.sh = (int)(first & 31);
    }
  };
  auto load = [&](Step& s, int step) {
    if ((step + 1) * kStep <= K) load_step(s, step * kStep, std::true_type{});      // (uniform)
    else load_step(s, step * kStep, std::false_type{});
  };
  // a step's lines into the wave's LDS; returns the signs of this lane's 16 k
  auto turn = [&](const Step& s) {
    wave_lds_fence();                                        // (the last step's reads are done)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int at = row_unit(8 * i + line, unit);
      *reinterpret_cast<float4*>(Xl + at) = s.x[i];
      if (HAS_RX) *reinterpret_cast<float4*>(RXl + at) = s.rx[i];
      *reinterpret_cast<float4*>(Yl + (Y_KC ? at : column_line(8 * i + line) + unit * 4)) = s.y[i];
    }
    uint32_t v = 0;
    if (HAS_V) {
      v = __builtin_amdgcn_alignbit(s.v1, s.v0, s.sh);
      if (!Y_KC && lhalf == 0) Vl[l32] = v;
    }
    wave_lds_fence();
    if (HAS_V && !Y_KC) {
      v = 0;
#pragma unroll
      for (int q = 0; q < kLane / 4; ++q) {
        const uint4 w = *reinterpret_cast<const uint4*>(Vl + lhalf * kLane + 4 * q);
        v |= ((w.x >> l32) & 1u) << (4 * q) | ((w.y >> l32) & 1u) << (4 * q + 1) | ((w.z >> l32) & 1u) << (4 * q + 2) | ((w.w >> l32) & 1u) << (4 * q + 3);
      }
    }
    return v;
  };
  // eight of a lane's k, from number h on: of row, column l32
  struct Operands { float x[8], rx[8], y[8]; };
  auto read8 = [&](Operands& o, int h) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int at = row_unit(l32, lhalf * 4 + (h >> 2) + q);
      auto get = [&](const float* l, float (&f)[8]) {
        const float4 t = *reinterpret_cast<const float4*>(l + at);
        f[4 * q] = t.x; f[4 * q + 1] = t.y; f[4 * q + 2] = t.z; f[4 * q + 3] = t.w;
      };
      get(Xl, o.x);
      if (HAS_RX) get(RXl, o.rx);
      if (Y_KC) {
        get(Yl, o.y);
      } else {
#pragma unroll
        for (int j = 4 * q; j < 4 * q + 4; ++j) o.y[j] = Yl[column_line(lhalf * kLane + h + j) + l32];
      }
    }
  };
  const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  floatx16 acc, racc, t, tr;
  auto multiply8 = [&](int h, uint32_t signs, auto whole) {
    Operands s;
    read8(s, h);
    bf16x8 v;
    if (HAS_V) {
      const uint32_t b = signs >> h;
      v = __builtin_bit_cast(bf16x8, make_uint4(sign_pair(b, b >> 1), sign_pair(b >> 2, b >> 3), sign_pair(b >> 4, b >> 5), sign_pair(b >> 6, b >> 7)));
    }
    if constexpr (decltype(whole)::value) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (HAS_C) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(s.x[j], s.y[j], acc, 0, 0, 0);
        if (HAS_RX) racc = __builtin_amdgcn_mfma_f32_32x32x2f32(s.rx[j], s.y[j], racc, 0, 0, 0);
        if (HAS_V) racc = __builtin_amdgcn_mfma_f32_32x32x2f32(s.x[j], (float)v[j] * (1.f / kScale), racc, 0, 0, 0);
      }
    } else {
      auto pieces = [&](const float (&f)[8], bf16x8 (&o)[3]) {
        uint32_t p[3][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) split_pair<false>(f[2 * q], f[2 * q + 1], p[0][q], p[1][q], p[2][q]);
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
  auto multiply = [&](uint32_t signs, auto whole) { multiply8(0, signs, whole); multiply8(8, signs, whole); };
  auto contract = [&](auto whole) {
    acc = zero; racc = zero; t = zero; tr = zero;
    Step s0, s1;
    const int n = wave < steps ? (steps - wave + NW - 1) / NW : 0;         // steps of this wave (uniform)
    if constexpr (decltype(whole)::value) {
      for (int i = 0; i < n; ++i) { load(s0, wave + i * NW); multiply(turn(s0), whole); }
    } else if (n == 1) {
      load(s0, wave);
      multiply(turn(s0), whole);
    } else if (n > 1) {
      // two steps in flight, and no condition between their loads: the wait for the older step then leaves the younger one's out
      load(s0, wave); load(s1, wave + NW);
      auto next = [&](Step& r, int i) {                      // step i of the wave, and ask for step i + 2
        const uint32_t signs = turn(r);
        load(r, wave + (i + 2) * NW);
        multiply(signs, whole);
      };
      int i = 0;
      for (; i + 3 < n; i += 2) { next(s0, i); next(s1, i + 1); }
      if (i + 2 < n) {                                       // three left
        next(s0, i);
        multiply(turn(s1), whole);
        multiply(turn(s0), whole);
      } else {
        multiply(turn(s0), whole);
        multiply(turn(s1), whole);
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
  __syncthreads();                                           // (the waves' regions of LDS)
  float* part = lds;
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
  constexpr int parts = ((FM != 1 ? 1 : 0) + (HAS_RX || HAS_V ? 1 : 0)) * kEdge * kEdge, turns = wave_floats(Y_KC, HAS_RX, HAS_V);
  constexpr int smem = NW * (parts > turns ? parts : turns) * (int)sizeof(float);
  auto kern = short_gemm_f32<NW, Y_KC, HAS_RX, HAS_V, EPI, FM>;
  if (smem > 64 * 1024) {
    static LdsLimitOnce lim;
    const hipError_t e = lim.raise(reinterpret_cast<const void*>(kern), smem);
    if (e != hipSuccess) return e;
  }
  const int64_t tiles = (int64_t)((a.M + kEdge - 1) / kEdge) * ((a.N + kEdge - 1) / kEdge);
  hipLaunchKernelGGL(kern, xcd_grid(tiles * active_count(a.active_mask, a.k)), dim3(NW * 64), smem, s, a);
  return hipGetLastError();
}

}  // namespace f32s

// A product of M x N outputs and contraction K for each of k workers (the layout asks as well: such a product needs no slices).
// Against the 64 x 64 tiles, in slices where there are few of them; times of a class of products a step, here / there, us.  `tiles`: the
// 64 x 64 ones of all workers; `blocks`: this kernel's, of which 256 run at a time.
//   tiles  256 and more fill the chip and share their operands among more outputs (512-1024, four of 256: the step 119 / 106)
//   K      up to 1152, forward: faster as a rule (128-128, two workers of 64: the step 38 / 74; 1036-340, five of 93: 75 / 92; but 100 -> 3200,
//          four of 64: 32 / 25)
//          up to 1152, data gradient: up to 512 blocks, two rounds (512 -> 2048, four of 64: 0.84 of the tiles' time; 64 -> 2048: 0.89), but
//          few blocks take too long over a long contraction (1024 -> 256, four of 64: 29.7 / 28.0; 768 -> 256: 0.92).  The third round
//          pays in the middle (256 -> 3072: 0.90; 140: 1.01; 10: 1.40; 768: 1.01), further ones don't (140 -> 3200: 39 / 34; 10 -> 3200: 1.41;
//          1024 -> 3200: 78 / 61).  Without the companion's products the third round takes 512 -> 3072: 0.94, 1024: 1.05, and short
//          contractions of up to 320 pay as a rule (64 -> 4000: 0.84; 256: 0.93; 140: 1.07; 512: 1.04, -> 3200 1.13)
//          longer: one round (2048 -> 1024, four of 64: 0.87, 2048 -> 1280: 1.18) that is not too empty (3072 -> 512: 1.13, 2048 -> 512: 1.03,
//          4096 -> 1024 0.95).  The first layer, which has no companion: 32 to 128 tiles (1280-256, six of 256, 96: the step 92 / 96;
//          2048 -> 2048, four of 64, 128: 0.85; 4096-64, one of 64, one: the step 61 / 48)
bool gemm_f32_short_shape(int64_t M, int64_t N, int64_t K, int k, ShortProduct what) {
  const int64_t tiles = ((M + 63) / 64) * ((N + 63) / 64) * k, blocks = ((M + 31) / 32) * ((N + 31) / 32) * k;
  if (tiles >= 256) return false;
  if (K > 1152) {
    if (what == SHORT_FIRST) return K <= 4096 && tiles >= 32 && tiles <= 128;
    return tiles >= 32 && blocks <= 256 && K <= (tiles < 48 ? 2048 : 4096);
  }
  if (what != SHORT_GRAD && what != SHORT_PLAIN_GRAD) return true;
  const bool plain = what == SHORT_PLAIN_GRAD;
  if (blocks <= 512) return plain || blocks >= 128 || K <= 896;
  if (blocks <= 768) return K <= 640 && (plain || K >= 192);
  return plain && K <= 320;
}

// Forward product or data gradient of matrices in memory, no slices, whose 64 x 64 tiles over all workers would leave compute
// units idle.  (Whichever workers are active: the choice must not depend on who steps.)
bool gemm_f32_short_ok(const GemmArgs& a) {
  if (a.x_view != VIEW_NONE || a.y_view != VIEW_NONE || a.ksplit > 1 || !(a.ry_bits || a.plain)) return false;
  if (a.epi == EPI_MASK ? !a.plain && !a.RX : a.epi != EPI_RELU) return false;
  const ShortProduct what = a.epi == EPI_MASK ? (a.plain ? SHORT_PLAIN_GRAD : SHORT_GRAD) : a.plain ? SHORT_PLAIN : a.RX ? SHORT_LATER : SHORT_FIRST;
  return gemm_f32_short_shape(a.M, a.N, a.K, a.k, what);
}

template <int NW>
static hipError_t launch_short(const GemmArgs& a, hipStream_t s) {
  using namespace f32s;
  if (a.epi == EPI_MASK) {
    if (a.plain) return launch<NW, false, false, false, EPI_MASK, 0>(a, s);
    return a.r_only ? launch<NW, false, true, true, EPI_MASK, 1>(a, s) : launch<NW, false, true, true, EPI_MASK, 0>(a, s);
  }
  const bool rx = a.RX != nullptr;
  if (a.plain) return launch<NW, true, false, false, EPI_RELU, 0>(a, s);
  if (a.r_only) return rx ? launch<NW, true, true, true, EPI_RELU, 1>(a, s) : launch<NW, true, false, true, EPI_RELU, 1>(a, s);
  return rx ? launch<NW, true, true, true, EPI_RELU, 0>(a, s) : launch<NW, true, false, true, EPI_RELU, 0>(a, s);
}

hipError_t launch_gemm_f32_short(const GemmArgs& a, hipStream_t s) {
  KernelScope ks(a.epi == EPI_MASK ? KC_GEMM_DGRAD : KC_GEMM_FWD, s);
  // (up to 64 k: a step each for two waves, or one for the first; the second then only helps to write the tile: 8.8 us, alone 11.0)
  return a.K > 2 * f32s::kStep ? launch_short<8>(a, s) : launch_short<2>(a, s);
}

}  // namespace dw
