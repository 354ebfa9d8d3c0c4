// fp32 "dual-number" GEMM for gfx950: C = X*Y and RC = RX*Y + X*RY in one pass over the tiles.
//
// Forward and backward propagation of the MLP (Section II eq.(2)) and the propagation of their
// directional derivatives along z, which yields the Hessian-vector product Hz of the Hutchinson estimate
// (Section IV-B), all have this product-rule shape:
//   forward      s  = a W^T,            Rs  = Ra W^T + a V^T            (V = z reshaped like W)
//   data grad    d' = d W,              Rd' = Rd W + d V
//   weight grad  gW = d^T a,            HzW = Rd^T a + d^T Ra
// so one kernel template serves the three, sharing every tile load between the plain product and its
// R-companion.  The +-1 operand V is never stored as a matrix: its tile is expanded from the sign bits of
// z while the W tile is staged.
//
// The products run on the bf16 matrix cores, every float split into three pieces (dw_f32_pieces.h).  Contractions of one or two,
// and tiles whose results are not finite once more, run on the fp32 matrix instruction (below).
//
// Tiling: waves of 32 rows by 32 or 64 columns; tiles of 32 k are split into their pieces once per block while they are
// stored to LDS (planes [row][32 k] of bf16, 64-byte rows, 16-byte units XOR-swizzled so that both the
// reads of 8 consecutive rows and the stores of every fourth row spread over the banks); global loads are 16-byte and one
// tile ahead in registers.  On the fp32 matrix instruction -> now: eight workers, 256 samples, 3072-1024-1024-1024: forward
// 295 / 135 -> 147 / 74 us (first / later layers), data gradient 94 -> 59, fused weight gradients 346 / 154 -> 233 / 103; eight
// workers, 64 maps of 26 x 26 x 32 -> 24 x 24 x 64: weight gradient 370 -> 255 (forward 207 and data gradient 384 through
// this kernel's views of the map, 166 and 187 on slabs of it, dw_conv_f32.hip, which takes all maps whose slabs fit in LDS).
// What bounds them now (64 x 64 and 64 x 128 tiles of the first, by counters): matrix cores 30 to 36 % busy, vector arithmetic
// (splitting, 6.5 instructions per element and block that loads it) 36 to 45 %, LDS instructions 40 to 47 % (six bytes stored and
// read per element), and between them the two barriers a tile, with two blocks a compute unit to hide them; the convolutions
// 20 to 38 %, 41 to 49 % and 31 to 56 %.  Two tiles in flight instead of one: no change.
#include <cstddef>
#include <type_traits>

#include "dw_internal.h"
#include "dw_f32_pieces.h"
#include "dw_fused_update.h"

namespace dw {

constexpr int BK = 32;                     // k per tile
constexpr int kRowBytes = 64;              // of a plane

enum RyMode { RY_NONE = 0, RY_MEM = 1, RY_BITS = 2 };

// byte offset inside a plane of the 16-byte unit holding k = 8*oct .. 8*oct+7 of `row`: four rows share the 256 bytes that
// the 64 banks serve at once, and the unit's place in them is XORed with the group's number, so that 16 consecutive rows
// (operand reads), 4 rows with their 4 units (stores, k contiguous) and every fourth row of 64 (stores, k-major) all
// use 16 different places
__device__ __forceinline__ int unit_at(int row, int oct) {
  const int m = row >> 2;
  return m * 256 + ((((row & 3) * 4 + oct) ^ (m & 15)) << 4);
}

// Loads the tiles of one operand (NOPS = 1) or of an operand and its R-companion, laid out alike (NOPS = 2), and stores
// their pieces.  A unit of work is 8 consecutive k of one row when k is contiguous in memory (KC), else 4 k of 4 consecutive rows.
// Rows past the end repeat the last ones (their results are never stored); k past the end is zero.
// VIEW: OperandView, the operand is read out of a map.
template <int NT, int ROWS, bool KC, int NOPS, int VIEW>
struct TileLoader {
  static constexpr int PER = KC ? ROWS * 4 : ROWS * 2;       // units per operand
  static constexpr int NU = (PER * NOPS + NT - 1) / NT;
  static constexpr int NV = KC ? 2 : 4;                      // float4 per unit
  static constexpr int PLANE = ROWS * kRowBytes;

  using Pieces = uint32_t[NU][3][NV * 2];                    // in pairs: k by k (KC), or row by row
  float4 v[NU][NV];                                          // the tile on its way from memory
  const float* p[NU];                                        // KC: the unit's row; else its four rows at k = 0
  int a0[NU], a1[NU];                                        // views: what the unit keeps about its row or its k
  int ld; uint32_t magic;
  ConvView cv;

  __device__ __forceinline__ static bool unit(int u, int t, int& op, int& w) {
    const int idx = u * NT + t;
    op = NOPS == 2 ? idx / PER : 0;
    w = idx - op * PER;
    return NU * NT == PER * NOPS || idx < PER * NOPS;
  }

  // t: the thread's place among the loader's; r0, R: first row of the tile and rows of the operand
  __device__ __forceinline__ void begin(const float* src, const float* rsrc, int ld_, int r0, int R, int kbeg, const ConvView& c, int t) {
    ld = ld_; cv = c;
    if (VIEW != VIEW_NONE) magic = 0xFFFFFFFFu / (uint32_t)(VIEW == VIEW_PATCH ? c.Cin : c.Cout) + 1u;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      int op, w;
      if (!unit(u, t, op, w)) { op = 0; w = 0; }
      const float* s = op ? rsrc : src;
      if (KC) {
        const int row = r0 + (w >> 2) < R ? r0 + (w >> 2) : R - 1;
        if (VIEW == VIEW_PATCH) {
          const int Wo = c.W - 2, Ho = c.H - 2;
          const int x = row % Wo, tt = row / Wo, y = tt % Ho, b = tt / Ho;
          p[u] = s + (((int64_t)b * c.H + y) * c.W + x) * c.Cin;
        } else if (VIEW == VIEW_SHIFTED) {
          const int xx = row % c.W, tt = row / c.W, yy = tt % c.H, b = tt / c.H;
          p[u] = s + (int64_t)b * (c.H - 2) * (c.W - 2) * c.Cout;
          a0[u] = yy; a1[u] = xx;
        } else {
          p[u] = s + (int64_t)row * ld + (w & 3) * 8;
        }
      } else {
        const int rg = w % (ROWS / 4), last = (R - 1) & ~3;
        const int r = r0 + rg * 4 < R ? r0 + rg * 4 : last;
        if (VIEW == VIEW_PATCH) {                            // r is a column of the patch matrix: a tap and a channel
          const int tap = (int)__umulhi((uint32_t)r, magic), ci = r - tap * c.Cin, dy = (tap * 11) >> 5, dx = tap - dy * 3;
          p[u] = s + ((int64_t)dy * c.W + dx) * c.Cin + ci;
          // the position of the unit's first k: row of the map (over all images) and column
          const int pos = kbeg + (w / (ROWS / 4)) * 4, Wo = c.W - 2, Ho = c.H - 2;
          const int x = pos % Wo, tt = pos / Wo, y = tt % Ho, b = tt / Ho;
          a0[u] = b * c.H + y; a1[u] = x | (y << 16);
        } else {
          p[u] = s + r;
        }
      }
    }
  }

  // the tile at k0; called for k0 = kbeg, kbeg + BK, ... in order
  // WHOLE: no k of the tile is past the end
  template <bool WHOLE>
  __device__ __forceinline__ void load(int k0, int kend, int t) {
    const bool whole = WHOLE || k0 + BK <= kend;             // (uniform)
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      int op, w;
      if (!unit(u, t, op, w)) continue;
      const int kk = k0 + (KC ? (w & 3) * 8 : (w / (ROWS / 4)) * 4);
      if (KC) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int k = kk + q * 4;
          bool ok = whole || k < kend;
          const float* a;
          if (VIEW == VIEW_PATCH) {
            const int tap = (int)__umulhi((uint32_t)k, magic), ci = k - tap * cv.Cin, dy = (tap * 11) >> 5, dx = tap - dy * 3;
            a = p[u] + (dy * cv.W + dx) * cv.Cin + ci;
          } else if (VIEW == VIEW_SHIFTED) {
            const int tap = (int)__umulhi((uint32_t)k, magic), co = k - tap * cv.Cout, dy = (tap * 11) >> 5, dx = tap - dy * 3;
            const int y = a0[u] - dy, x = a1[u] - dx;
            ok = ok && y >= 0 && y < cv.H - 2 && x >= 0 && x < cv.W - 2;
            a = p[u] + ((int64_t)y * (cv.W - 2) + x) * cv.Cout + co;
          } else {
            a = p[u] + k0 + q * 4;
          }
          v[u][q] = ok ? *reinterpret_cast<const float4*>(a) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
      } else if (VIEW == VIEW_PATCH) {
        int x = a1[u] & 0xFFFF, y = a1[u] >> 16, row = a0[u];
        const int Wo = cv.W - 2, Ho = cv.H - 2;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool ok = whole || kk + j < kend;
          v[u][j] = ok ? *reinterpret_cast<const float4*>(p[u] + ((int64_t)row * cv.W + x) * cv.Cin) : make_float4(0.f, 0.f, 0.f, 0.f);
          if (j < 3 && ++x == Wo) { x = 0; ++row; if (++y == Ho) { y = 0; row += 2; } }
        }
        x = (a1[u] & 0xFFFF) + BK; y = a1[u] >> 16; row = a0[u];
        while (x >= Wo) { x -= Wo; ++row; if (++y == Ho) { y = 0; row += 2; } }
        a0[u] = row; a1[u] = x | (y << 16);
      } else {
        const float* a;
        int64_t step;
        if (VIEW == VIEW_TAPS) {                             // four channels of one tap (channel counts are multiples of 4)
          const int tap = (int)__umulhi((uint32_t)kk, magic), co = kk - tap * cv.Cout;
          step = 9 * cv.Cin;
          a = p[u] + co * step + tap * cv.Cin;
        } else {
          step = ld;
          a = p[u] + kk * step;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
          v[u][j] = (whole || kk + j < kend) ? *reinterpret_cast<const float4*>(a + j * step) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
  }

  // unit u of v into its pieces.  sums: [NU][4], receives the column sums of the unit's rows (k-major operands; bias
  // gradients)
  template <bool HALVES>
  __device__ __forceinline__ void split_unit(int u, uint32_t (&s)[3][NV * 2], bool want_sums, float (&sums)[NU][4]) const {
    if constexpr (KC) {
      const float x[8] = {v[u][0].x, v[u][0].y, v[u][0].z, v[u][0].w, v[u][1].x, v[u][1].y, v[u][1].z, v[u][1].w};
      split_pairs<HALVES, 4>(x, s);
    } else {
      const float x[16] = {v[u][0].x, v[u][1].x, v[u][2].x, v[u][3].x, v[u][0].y, v[u][1].y, v[u][2].y, v[u][3].y,
                           v[u][0].z, v[u][1].z, v[u][2].z, v[u][3].z, v[u][0].w, v[u][1].w, v[u][2].w, v[u][3].w};
      if (want_sums) {
#pragma unroll
        for (int r = 0; r < 4; ++r) sums[u][r] += (x[4 * r] + x[4 * r + 1]) + (x[4 * r + 2] + x[4 * r + 3]);
      }
      split_pairs<HALVES, 8>(x, s);
    }
  }
  __device__ __forceinline__ static void store_unit(char* lds, int op, int w, const uint32_t (&s)[3][NV * 2]) {
    char* base = lds + op * 3 * PLANE;
    if constexpr (KC) {
      char* at = base + unit_at(w >> 2, w & 3);
#pragma unroll
      for (int c = 0; c < 3; ++c) *reinterpret_cast<uint4*>(at + c * PLANE) = make_uint4(s[c][0], s[c][1], s[c][2], s[c][3]);
    } else {
      const int rg = w % (ROWS / 4), kq = w / (ROWS / 4);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        char* at = base + unit_at(rg * 4 + r, kq >> 1) + (kq & 1) * 8;
#pragma unroll
        for (int c = 0; c < 3; ++c) *reinterpret_cast<uint2*>(at + c * PLANE) = make_uint2(s[c][2 * r], s[c][2 * r + 1]);
      }
    }
  }
  // the two together, unit by unit
  template <bool HALVES>
  __device__ __forceinline__ void split_store(char* lds, int t, bool want_sums, float (&sums)[NU][4]) const {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      int op, w;
      if (!unit(u, t, op, w)) continue;
      uint32_t s[3][NV * 2];
      split_unit<HALVES>(u, s, want_sums, sums);
      store_unit(lds, op, w, s);
    }
  }
};

// The same units for the +-1 operand: sign bits in, one plane of bf16 out.  k past the end need not be zero (the other
// operand's is); its bits are not read.
template <int NT, int ROWS, bool KC, int VIEW>
struct SignLoader {
  static constexpr int PER = KC ? ROWS * 4 : ROWS * 2;
  static constexpr int NU = (PER + NT - 1) / NT;
  uint32_t b[NU];                                            // KC: 8 bits; else 4 x 4 bits, k by k
  int64_t p[NU];                                             // bit offset: KC the unit's row; else its rows at k = 0
  int ld; uint32_t magic; ConvView cv;

  __device__ __forceinline__ void begin(int64_t z_off, int ld_, int r0, int R, const ConvView& c, int t) {
    ld = ld_; cv = c;
    if (VIEW == VIEW_TAPS) magic = 0xFFFFFFFFu / (uint32_t)c.Cout + 1u;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int w = u * NT + t < PER ? u * NT + t : 0;
      if (KC) {
        const int row = r0 + (w >> 2) < R ? r0 + (w >> 2) : R - 1;
        p[u] = z_off + (int64_t)row * ld;
      } else {
        const int rg = w % (ROWS / 4);
        p[u] = z_off + (r0 + rg * 4 < R ? r0 + rg * 4 : (R - 1) & ~3);
      }
    }
  }
  __device__ __forceinline__ void load(const uint32_t* zb, int k0, int kend, int t) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int w = u * NT + t;
      if (NU * NT != PER && w >= PER) continue;
      if (KC) {
        const int k = k0 + (w & 3) * 8;
        // two groups of four bits (K is a multiple of 4, so a group lies in one word)
        const int64_t o0 = p[u] + (k < kend ? k : kend - 4), o1 = p[u] + (k + 4 < kend ? k + 4 : kend - 4);
        b[u] = ((zb[o0 >> 5] >> (o0 & 31)) & 0xFu) | (((zb[o1 >> 5] >> (o1 & 31)) & 0xFu) << 4);
      } else {
        const int k = k0 + (w / (ROWS / 4)) * 4;
        uint32_t x = 0;
        int64_t o, step;
        if (VIEW == VIEW_TAPS) {
          const int kc = k < kend ? k : kend - 4;
          const int tap = (int)__umulhi((uint32_t)kc, magic), co = kc - tap * cv.Cout;
          step = 9 * cv.Cin;
          o = p[u] + co * step + tap * cv.Cin;
#pragma unroll
          for (int j = 0; j < 4; ++j) { const int64_t q = o + j * step; x |= ((zb[q >> 5] >> (q & 31)) & 0xFu) << (4 * j); }
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int64_t q = p[u] + (int64_t)(k + j < kend ? k + j : kend - 1) * ld;
            x |= ((zb[q >> 5] >> (q & 31)) & 0xFu) << (4 * j);
          }
        }
        b[u] = x;
      }
    }
  }
  __device__ __forceinline__ void store(char* lds, int t) const {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int w = u * NT + t;
      if (NU * NT != PER && w >= PER) continue;
      const uint32_t x = b[u];
      if (KC) {
        *reinterpret_cast<uint4*>(lds + unit_at(w >> 2, w & 3)) =
            make_uint4(sign_pair(x, x >> 1), sign_pair(x >> 2, x >> 3), sign_pair(x >> 4, x >> 5), sign_pair(x >> 6, x >> 7));
      } else {
        const int rg = w % (ROWS / 4), kq = w / (ROWS / 4);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          *reinterpret_cast<uint2*>(lds + unit_at(rg * 4 + r, kq >> 1) + (kq & 1) * 8) =
              make_uint2(sign_pair(x >> r, x >> (4 + r)), sign_pair(x >> (8 + r), x >> (12 + r)));
      }
    }
  }
};

// rows of 64 bytes the operand planes take: three per element and operand, one for signs
constexpr int gemm_f32_rows(int bm, int bn, bool has_rx, int rym) {
  return 3 * bm * (has_rx ? 2 : 1) + 3 * bn * (rym == RY_MEM ? 2 : 1) + (rym == RY_BITS ? bn : 0);
}
constexpr int gemm_f32_lds(int bm, int bn, int wm, int wn, bool has_rx, int rym, int epi) {
  const int tiles = gemm_f32_rows(bm, bn, has_rx, rym) * kRowBytes;
  const int upd = epi == EPI_WGRAD_FUSED ? wm * wn * fused_update_lds_floats() * 4 : 0;    // the epilogue reuses the space
  return tiles > upd ? tiles : upd;
}

// the same on the fp32 matrix instruction, from the two halves of the numbers
__device__ __forceinline__ float joined(const bf16x8 (&x)[3], int j) {
  const u16x8 high = __builtin_bit_cast(u16x8, x[0]), low = __builtin_bit_cast(u16x8, x[1]);
  return __uint_as_float((uint32_t)high[j] << 16 | low[j]);
}
__device__ __forceinline__ void mfma_whole(const bf16x8 (&x)[3], const bf16x8 (&y)[3], floatx16& t) {
#pragma unroll
  for (int j = 0; j < 8; ++j) t = __builtin_amdgcn_mfma_f32_32x32x2f32(joined(x, j), joined(y, j), t, 0, 0, 0);
}
__device__ __forceinline__ void mfma_whole(const bf16x8 (&x)[3], const bf16x8& v, floatx16& t) {
#pragma unroll
  for (int j = 0; j < 8; ++j) t = __builtin_amdgcn_mfma_f32_32x32x2f32(joined(x, j), (float)v[j] * (1.f / kScale), t, 0, 0, 0);
}

// XV, YV: OperandView of X/RX and of Y/RY (convolutions without a patch matrix in memory).  FM == 1: a Hutchinson probe
// other than the step's last (fused) or first (forward, data gradient): the R-products alone.
template <int BM, int BN, int WM, int WN, bool X_KC, bool Y_KC, bool HAS_RX, int RYM, int EPI, int FM = 0, int XV = VIEW_NONE,
          int YV = VIEW_NONE>
__global__ __launch_bounds__(WM * WN * 64, 2) void dual_gemm_f32(GemmArgs a) {
  constexpr int NT = WM * WN * 64;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  static_assert(TM >= 1 && TN >= 1, "wave tile must hold at least one 32x32 MFMA tile");
  constexpr bool HAS_C = FM != 1;                            // the plain product is computed
  constexpr bool HAS_R = HAS_RX || RYM != RY_NONE;           // the R-companion is
  constexpr bool STAGED = X_KC && Y_KC && BM == 64 && BN == 64;
  // consecutive blocks of an XCD: the row tiles of a column tile (its W panel is read once), then the next column tile, the next slice,
  // the next worker
  const unsigned tiles_m = (a.M + BM - 1) / BM, tiles = tiles_m * ((a.N + BN - 1) / BN);
  const unsigned slices = a.ksplit > 1 ? a.ksplit : 1, logical = xcd_unit(), slot = logical / (tiles * slices);
  if (slot >= (unsigned)active_count(a.active_mask, a.k)) return;
  const int worker = nth_active_worker(a.active_mask, slot);
  const unsigned in_worker = logical - slot * (tiles * slices), in_slice = in_worker % tiles;
  const int slice = in_worker / tiles, tm = in_slice % tiles_m, tn = in_slice / tiles_m;
  const int row0 = tm * BM, col0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave % WM) * (BM / WM), wn0 = (wave / WM) * (BN / WN);
  const int l32 = lane & 31, lhalf = lane >> 5;

  extern __shared__ __attribute__((aligned(16))) char lds[];
  using LX = TileLoader<NT, BM, X_KC, HAS_RX ? 2 : 1, XV>;
  using LY = TileLoader<NT, BN, Y_KC, RYM == RY_MEM ? 2 : 1, YV>;
  using LS = SignLoader<NT, BN, Y_KC, YV>;
  char* Xl = lds;
  char* Yl = Xl + 3 * (HAS_RX ? 2 : 1) * LX::PLANE;
  char* Sl = Yl + 3 * LY::PLANE;                             // signs, or the planes of RY

  const float* X = reinterpret_cast<const float*>(a.X) + (int64_t)worker * a.x_wstride;
  const float* RX = HAS_RX ? reinterpret_cast<const float*>(a.RX) + (int64_t)worker * a.x_wstride : nullptr;
  const float* Y = reinterpret_cast<const float*>(a.Y) + (int64_t)worker * a.y_wstride;
  const float* RY = RYM == RY_MEM ? reinterpret_cast<const float*>(a.RY) + (int64_t)worker * a.y_wstride : nullptr;
  const uint32_t* zb = a.zbits + (int64_t)worker * a.z_stride;

  // the slice of the contraction this block covers (all of it unless the product is cut along k)
  const bool sliced = (EPI == EPI_WGRAD || EPI == EPI_RELU || EPI == EPI_MASK) && a.ksplit > 1;
  const int kchunk = sliced ? ((a.K + a.ksplit - 1) / a.ksplit + BK - 1) / BK * BK : a.K;
  const int kbeg = sliced ? slice * kchunk : 0;
  const int kend = sliced ? (kbeg + kchunk < a.K ? kbeg + kchunk : a.K) : a.K;
  const int nkt = kend > kbeg ? (kend - kbeg + BK - 1) / BK : 0;

  // acc, racc: the chains of the first pieces' products, then the results; t, tr: those of the others
  floatx16 acc[TM][TN], racc[TM][TN], t[TM][TN], tr[TM][TN];
  const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  LX lx; LY ly; LS ls;
  // a k-major Y that keeps half the block busy leaves the signs to the other half
  constexpr int S0 = RYM == RY_BITS && LY::PER * 2 == NT && LS::PER * 2 == NT ? NT / 2 : 0;
  const int ts = S0 ? (tid + NT - S0) % NT : tid;
  constexpr bool SUMS = EPI == EPI_WGRAD || EPI == EPI_WGRAD_FUSED;      // bias gradients: column sums of X and RX
  const bool want_sums = SUMS && tn == 0;
  float sums[LX::NU][4], none[LY::NU][4];

  // this lane's unit of k-step 0 in row l32 of each tile; k-step 1 is 32 bytes further under the swizzle
  int xat[TM], yat[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) xat[i] = unit_at(wm0 + i * 32 + l32, lhalf);
#pragma unroll
  for (int j = 0; j < TN; ++j) yat[j] = unit_at(wn0 + j * 32 + l32, lhalf);

  auto fetch = [&](int kt, auto whole) {
    const int k0 = kbeg + kt * BK;
    lx.template load<decltype(whole)::value>(k0, kend, tid);
    ly.template load<decltype(whole)::value>(k0, kend, tid);
    if (RYM == RY_BITS && !STAGED) ls.load(zb, k0, kend, ts);
  };
  auto fetch_signs = [&](int kt) { if (RYM == RY_BITS) ls.load(zb, kbeg + kt * BK, kend, ts); };   // (one tile ahead of the products)
  typename LX::Pieces xs;                                    // STAGED: the pieces of the next tile
  typename LY::Pieces ys;
  auto split = [&](auto halves) {
#pragma unroll
    for (int u = 0; u < LX::NU; ++u) lx.template split_unit<decltype(halves)::value>(u, xs[u], want_sums, sums);
#pragma unroll
    for (int u = 0; u < LY::NU; ++u) ly.template split_unit<decltype(halves)::value>(u, ys[u], false, none);
  };
  // Tile kt: its pieces go to LDS, then its products run.  STAGED (64 x 64 tiles of k-contiguous operands): the next tile
  // has arrived meanwhile, is split into pieces while the products run, and the one after it is asked for.  MAIN: that
  // one exists and is whole, so the step is straight-line code and the splitting is issued between the multiplies (forward,
  // 1024 wide: 92 -> 75 us).  Otherwise the next tile is asked for before the products and split after them: k-major
  // operands and larger tiles have no registers for the pieces (spills, half the speed).
  auto step = [&](int kt, auto main, auto halves) {
    constexpr bool MAIN = decltype(main)::value;
    constexpr bool HALVES = decltype(halves)::value;
    if constexpr (STAGED) {
#pragma unroll
      for (int u = 0; u < LX::NU; ++u) {
        int op, w;
        if (LX::unit(u, tid, op, w)) LX::store_unit(Xl, op, w, xs[u]);
      }
#pragma unroll
      for (int u = 0; u < LY::NU; ++u) {
        int op, w;
        if (LY::unit(u, tid, op, w)) LY::store_unit(Yl, op, w, ys[u]);
      }
    } else {
      lx.template split_store<HALVES>(Xl, tid, want_sums, sums);
      ly.template split_store<HALVES>(Yl, tid, false, none);
    }
    if (RYM == RY_BITS) ls.store(Sl, ts);
    __syncthreads();
    if (!STAGED) {
      if (kt + 1 < nkt) fetch(kt + 1, std::false_type{});
    } else if (MAIN || kt + 1 < nkt) {
      split(halves);
      fetch_signs(kt + 1);
      if (MAIN) fetch(kt + 2, std::true_type{});
      else if (kt + 2 < nkt) fetch(kt + 2, std::false_type{});
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      bf16x8 x[TM][3], rx[TM][3], y[TN][3], ry[TN][3];
      auto piece = [](const char* at) { return *reinterpret_cast<const bf16x8*>(at); };
#pragma unroll
      for (int c = 0; c < 3; ++c) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          x[i][c] = piece(Xl + c * LX::PLANE + (xat[i] ^ (s * 32)));
          if (HAS_RX) rx[i][c] = piece(Xl + (3 + c) * LX::PLANE + (xat[i] ^ (s * 32)));
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          if (HAS_C || HAS_RX) y[j][c] = piece(Yl + c * LY::PLANE + (yat[j] ^ (s * 32)));
          if (RYM == RY_MEM || (RYM == RY_BITS && c == 0)) ry[j][c] = piece(Sl + c * LY::PLANE + (yat[j] ^ (s * 32)));
        }
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          if constexpr (HALVES) {
            if (HAS_C) mfma_whole(x[i], y[j], acc[i][j]);
            if (HAS_RX) mfma_whole(rx[i], y[j], racc[i][j]);
            if (RYM == RY_MEM) mfma_whole(x[i], ry[j], racc[i][j]);
            if (RYM == RY_BITS) mfma_whole(x[i], ry[j][0], racc[i][j]);
          } else {
            if (HAS_C) mfma6(x[i], y[j], acc[i][j], t[i][j]);
            if (HAS_RX) mfma6(rx[i], y[j], racc[i][j], tr[i][j]);
            if (RYM == RY_MEM) mfma6(x[i], ry[j], racc[i][j], tr[i][j]);
            if (RYM == RY_BITS) mfma3(x[i], ry[j][0], racc[i][j], tr[i][j]);
          }
        }
    }
    __syncthreads();
  };
  // the whole contraction; returns whether a result is not finite
  auto contract = [&](auto with_main, auto halves) {
    lx.begin(X, RX, a.ldx, row0, a.M, kbeg, a.cv, tid);
    ly.begin(Y, RY, a.ldy, col0, a.N, kbeg, a.cv, tid);
    if (RYM == RY_BITS) ls.begin(a.z_off, a.ldy, col0, a.N, a.cv, ts);
#pragma unroll
    for (int u = 0; u < LX::NU; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) sums[u][r] = 0.f;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) { acc[i][j] = zero; racc[i][j] = zero; t[i][j] = zero; tr[i][j] = zero; }
    if (nkt > 0) fetch(0, std::false_type{});
    if (STAGED) {
      if (nkt > 0) { fetch_signs(0); split(halves); }
      if (nkt > 1) fetch(1, std::false_type{});
    }
    int kt = 0;
    if (STAGED && decltype(with_main)::value)
      for (; kbeg + (kt + 3) * BK <= kend; ++kt) step(kt, std::true_type{}, halves);
    for (; kt < nkt; ++kt) step(kt, std::false_type{}, halves);
    bool finite = true;
    if constexpr (!decltype(halves)::value) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          if (HAS_C) finite &= join_chains(acc[i][j], t[i][j]);
          if (HAS_R) finite &= join_chains(racc[i][j], tr[i][j]);
        }
    }
    return !finite;
  };
  // should a result not be finite, the block starts over with the fp32 matrix instruction on whole numbers; so does every block of a
  // very short contraction (asked after the pieces' pass: asked before it, what both passes share goes to scratch, fused weight
  // gradients 5 % slower)
  const bool again = __syncthreads_or(contract(std::true_type{}, std::false_type{}));
  if (again | (a.K < kWholeBelow)) contract(std::false_type{}, std::true_type{});

  if constexpr (SUMS) {
    // the units of a row lie with eight threads, 4 k each: their sums are added in order of k (the loop's last barrier is
    // behind the last read of the tiles)
    if (tn == 0) {
      float* part = reinterpret_cast<float*>(lds);           // [operand][8][BM]
#pragma unroll
      for (int u = 0; u < LX::NU; ++u) {
        int op, w;
        if (!LX::unit(u, tid, op, w)) continue;
        const int rg = w % (BM / 4), kq = w / (BM / 4);
#pragma unroll
        for (int r = 0; r < 4; ++r) part[(op * 8 + kq) * BM + rg * 4 + r] = sums[u][r];
      }
      __syncthreads();
      const int m = row0 + tid;
      if (tid < BM && m < a.M) {
        float gb = 0.f, hzb = 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          gb += part[q * BM + tid];
          if (HAS_RX) hzb += part[(8 + q) * BM + tid];
        }
        if (sliced) {
          float* pb = a.part_b + (((int64_t)slice * a.k + worker) * 2) * a.M;
          pb[m] = gb;
          if (HAS_RX) pb[a.M + m] = hzb;
        } else {
          a.gb[(int64_t)worker * a.c_wstride + m] = gb;
          if (HAS_RX) a.hzb[(int64_t)worker * a.c_wstride + m] = hzb;
        }
      }
      __syncthreads();
    }
  }

  if constexpr (EPI == EPI_WGRAD_FUSED) {
    // The update of Section IV-B applied to the tile instead of storing gW and HzW (see dw_fused_update.h): whole
    // tiles, wave tiles of 32 x 64; a private LDS region per wave where the operand tiles were.
    static_assert(TN == 2, "waves of 64 columns");
    float* fused_lds = reinterpret_cast<float*>(lds);
    const FuseArgs& f = a.fu;
    typedef const char __attribute__((address_space(4)))* karg_bytes;
    typedef const float __attribute__((address_space(4)))* karg_floats;
    const karg_bytes ka = (karg_bytes)__builtin_amdgcn_kernarg_segment_ptr();
    const karg_floats bc = (karg_floats)(ka + offsetof(GemmArgs, fu) + offsetof(FuseArgs, sc));
    const float ib1 = bc[worker], ib2 = bc[DW_MAX_K + worker];    // scalar loads from the kernel-argument block
    static_assert(offsetof(UpdateScalars, inv_bc2) == DW_MAX_K * sizeof(float), "inv_bc2 follows inv_bc1");
    // FM: 0 one Hutchinson probe; 1 a probe before the last (only the running sum of z*Hz is written); 2 the last
    // of several probes
    float nsum = 0.f;
    if constexpr (FM == 1)
      fused_probe_sum_wave_tile<TM>(racc, fused_lds + wave * fused_update_lds_floats(), f, (int64_t)worker * a.c_wstride,
                                    a.ldc, row0 + wm0, col0 + wn0, zb + (a.z_off >> 5), lane);
    else {
      FusedUpdateTile<TM, false, FM == 2 ? 1 : 0> upd(f, (int64_t)worker * a.c_wstride, a.ldc, row0 + wm0, col0 + wn0,
                                                     zb + (a.z_off >> 5), nullptr, lane);
      nsum = upd.run(acc, racc, racc, fused_lds + wave * fused_update_lds_floats(), ib1, ib2);
    }
    double ws = (double)nsum;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) ws += __shfl_xor(ws, off);
    __shared__ double red[NT / 64];
    if (lane == 0) red[wave] = ws;
    __syncthreads();
    if (tid == 0 && f.dist) {
      double sum = 0.0;
#pragma unroll
      for (int w = 0; w < NT / 64; ++w) sum += red[w];
      // one slot per 128 x 128 of W, cleared before the step: two blocks add to it, and 0 + p + q is 0 + q + p
      const int slot = row0 / 128 * (a.N / 128) + col0 / 128;
      static_assert(EPI != EPI_WGRAD_FUSED || (128 % BM == 0 && 128 / BM <= 2 && BN == 128), "at most two blocks to a slot");
      __hip_atomic_fetch_add(&f.partials[(int64_t)worker * f.part_stride + f.part_base + slot], sum, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
    }
    return;
  }
  // epilogue: lane holds column n = l32 of each 32x32 tile, rows (r/4)*8 + lhalf*4 + r%4
  float* C = reinterpret_cast<float*>(a.C) + (int64_t)worker * a.c_wstride;
  float* RC = reinterpret_cast<float*>(a.RC) + (int64_t)worker * a.c_wstride;
  if (sliced) {
    C = a.part + (((int64_t)slice * a.k + worker) * 2) * a.part_stride;
    RC = C + a.part_stride;
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = col0 + wn0 + j * 32 + l32;
    const bool n_ok = n < a.N;
    float bias = 0.f, cz = 0.f;
    if (EPI == EPI_RELU && n_ok) {
      bias = a.bias[(int64_t)worker * a.bias_wstride + n];
      const int64_t bi = a.zb_off + n;
      if (HAS_R) cz = ((zb[bi >> 5] >> (bi & 31)) & 1u) ? 1.f : -1.f;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = row0 + wm0 + i * 32 + (r >> 2) * 8 + lhalf * 4 + (r & 3);
        if (!n_ok || m >= a.M) continue;
        float c = acc[i][j][r], rc = racc[i][j][r];
        const int64_t o = (int64_t)m * a.ldc + n;
        if (sliced) {                                 // raw partial products: the epilogue follows the sum of the slices
          C[o] = c;
          if (HAS_R) RC[o] = rc;
        } else if (EPI == EPI_RELU && FM == 1) {      // a later probe: the activation is in memory, only its R-companion is new
          RC[o] = C[o] > 0.f ? rc + cz : 0.f;
        } else if (EPI == EPI_RELU) {
          c += bias; rc += cz;
          const bool on = c > 0.f;
          C[o] = on ? c : 0.f;
          if (HAS_R) RC[o] = on ? rc : 0.f;
        } else if (EPI == EPI_MASK) {
          const float* msk = reinterpret_cast<const float*>(a.mask_src) + (int64_t)worker * a.mask_wstride;
          const bool on = msk[(int64_t)m * a.ld_mask + n] > 0.f;
          if (FM != 1) C[o] = on ? c : 0.f;           // (a later probe: the plain data gradient is in memory already)
          if (HAS_R) RC[o] = on ? rc : 0.f;
        } else {
          C[o] = c;
          if (HAS_R) RC[o] = rc;
        }
      }
    }
  }
}

// ---- weight gradients of all layers of a small MLP in one launch ------------------------------------------------------------
// gW_l = d_l^T a_{l-1}, HzW_l = Rd_l^T a_{l-1} + d_l^T Ra_{l-1} and the bias gradients as above, 64 x 64 tiles of W_l, the layers' tiles
// behind each other.  Each layer's product alone fills a fraction of the chip and lasts as long as its trips to memory; together they
// last hardly longer than the longest, and the host has one launch to make instead of a launch and two events a layer.  Two
// tiles of 32 samples are on their way while one is multiplied.  784-512-512-10, four workers of 128 samples: 24 us for the three
// layers (13 to 14 each, two of them beside the data gradients on a second stream, and 20 us of the host's time for its
// events); a wave per 32 x 32 tile with its operands straight from memory 29: four times the loads and twice the splitting.
namespace f32g {

constexpr int EDGE = 64, NT = 256;

struct Layer {
  const float* x; const float* rx;                           // d_l, Rd_l of worker 0 [B][ldx]
  const float* y; const float* ry;                           // a_{l-1}, Ra_{l-1} (nullptr: the input) [B][N]
  int64_t x_wstride, y_wstride, woff, boff;                  // offsets in a row of g and of hz
  int ldx, M, N, tiles_m, first;                             // W_l is [M][N]; its first tile
};
struct Args {
  Layer layer[DW_MAX_LAYERS];
  int n, tiles, B, workers;                                  // workers: the active ones
  float* g; float* hz; int64_t Pp;                           // [k][Pp]
  uint64_t active_mask;
};

template <bool HAS_R, bool HAS_RY>
__device__ __forceinline__ void run_tile(const Args& a, const Layer& y, int tile, int worker, char* lds) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, lhalf = lane >> 5;
  const int tm = tile % y.tiles_m, tn = tile / y.tiles_m, row0 = tm * EDGE, col0 = tn * EDGE;
  const int wm0 = (wave & 1) * 32, wn0 = (wave >> 1) * 32;
  using LX = TileLoader<NT, EDGE, false, HAS_R ? 2 : 1, VIEW_NONE>;
  using LY = TileLoader<NT, EDGE, false, HAS_RY ? 2 : 1, VIEW_NONE>;
  char* Xl = lds;
  char* Yl = Xl + 3 * (HAS_R ? 2 : 1) * LX::PLANE;
  const float* X = y.x + worker * y.x_wstride;
  const float* RX = HAS_R ? y.rx + worker * y.x_wstride : nullptr;
  const float* Y = y.y + worker * y.y_wstride;
  const float* RY = HAS_RY ? y.ry + worker * y.y_wstride : nullptr;
  const int K = a.B, nkt = (K + BK - 1) / BK;
  const int xat = unit_at(wm0 + l32, lhalf), yat = unit_at(wn0 + l32, lhalf);   // of k-step 0
  const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  floatx16 acc, racc, t, tr;
  float sums[LX::NU][4], none[LY::NU][4];
  const ConvView no_view{};

  auto contract = [&](auto halves) {
    constexpr bool HALVES = decltype(halves)::value;
    LX lx[2]; LY ly[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      lx[h].begin(X, RX, y.ldx, row0, y.M, 0, no_view, tid);
      ly[h].begin(Y, RY, y.N, col0, y.N, 0, no_view, tid);
    }
    acc = zero; racc = zero; t = zero; tr = zero;
#pragma unroll
    for (int u = 0; u < LX::NU; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) sums[u][r] = 0.f;
    auto fetch = [&](int h, int kt) {
      if ((kt + 1) * BK <= K) { lx[h].template load<true>(kt * BK, K, tid); ly[h].template load<true>(kt * BK, K, tid); }
      else { lx[h].template load<false>(kt * BK, K, tid); ly[h].template load<false>(kt * BK, K, tid); }
    };
    // FETCH: the tile after the next one exists and is asked for
    auto step = [&](auto which, int kt, auto fetch_next) {
      constexpr int h = decltype(which)::value;
      lx[h].template split_store<HALVES>(Xl, tid, tn == 0, sums);
      ly[h].template split_store<HALVES>(Yl, tid, false, none);
      __syncthreads();
      if constexpr (decltype(fetch_next)::value) fetch(h, kt + 2);
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        bf16x8 x[3], rx[3], yv[3], ry[3];
        auto piece = [](const char* at) { return *reinterpret_cast<const bf16x8*>(at); };
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          x[c] = piece(Xl + c * LX::PLANE + (xat ^ (s * 32)));
          yv[c] = piece(Yl + c * LY::PLANE + (yat ^ (s * 32)));
          if (HAS_R) rx[c] = piece(Xl + (3 + c) * LX::PLANE + (xat ^ (s * 32)));
          if (HAS_RY) ry[c] = piece(Yl + (3 + c) * LY::PLANE + (yat ^ (s * 32)));
        }
        if constexpr (HALVES) {
          mfma_whole(x, yv, acc);
          if (HAS_R) mfma_whole(rx, yv, racc);
          if (HAS_RY) mfma_whole(x, ry, racc);
        } else {
          mfma6(x, yv, acc, t);
          if (HAS_R) mfma6(rx, yv, racc, tr);
          if (HAS_RY) mfma6(x, ry, racc, tr);
        }
      }
      __syncthreads();
    };
    using Even = std::integral_constant<int, 0>;
    using Odd = std::integral_constant<int, 1>;
    fetch(0, 0);
    if (nkt > 1) fetch(1, 1);
    int kt = 0;
    for (; kt + 3 < nkt; kt += 2) {
      step(Even{}, kt, std::true_type{});
      step(Odd{}, kt + 1, std::true_type{});
    }
    if (kt + 2 < nkt) {                                      // three left
      step(Even{}, kt, std::true_type{});
      step(Odd{}, kt + 1, std::false_type{});
      step(Even{}, kt + 2, std::false_type{});
    } else {
      step(Even{}, kt, std::false_type{});
      if (kt + 1 < nkt) step(Odd{}, kt + 1, std::false_type{});
    }
    bool finite = true;
    if constexpr (!HALVES) {
      finite &= join_chains(acc, t);
      if (HAS_R) finite &= join_chains(racc, tr);
    }
    return !finite;
  };
  const bool again = __syncthreads_or(contract(std::false_type{}));      // (see dual_gemm_f32)
  if (again | (K < kWholeBelow)) contract(std::true_type{});

  float* g = a.g + worker * a.Pp;
  float* hz = a.hz + worker * a.Pp;
  if (tn == 0) {                                             // bias gradients: the sums of eight threads, in order of k
    float* part = reinterpret_cast<float*>(lds);             // [operand][8][EDGE]
#pragma unroll
    for (int u = 0; u < LX::NU; ++u) {
      int op, w;
      if (!LX::unit(u, tid, op, w)) continue;
      const int rg = w % (EDGE / 4), kq = w / (EDGE / 4);
#pragma unroll
      for (int r = 0; r < 4; ++r) part[(op * 8 + kq) * EDGE + rg * 4 + r] = sums[u][r];
    }
    __syncthreads();
    const int m = row0 + tid;
    if (tid < EDGE && m < y.M) {
      float gb = 0.f, hzb = 0.f;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        gb += part[q * EDGE + tid];
        if (HAS_R) hzb += part[(8 + q) * EDGE + tid];
      }
      g[y.boff + m] = gb;
      if (HAS_R) hz[y.boff + m] = hzb;
    }
  }
  const int n = col0 + wn0 + l32;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = row0 + wm0 + (r >> 2) * 8 + lhalf * 4 + (r & 3);
    if (n >= y.N || m >= y.M) continue;
    const int64_t o = y.woff + (int64_t)m * y.N + n;
    g[o] = acc[r];
    if (HAS_R) hz[o] = racc[r];
  }
}

// PLAIN: a first-order step, g alone
template <bool PLAIN>
__global__ __launch_bounds__(NT, 2) void wgrad_group_f32(Args a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const unsigned logical = xcd_unit(), slot = logical / (unsigned)a.tiles;
  if (slot >= (unsigned)a.workers) return;
  const int worker = nth_active_worker(a.active_mask, slot), t = logical - slot * a.tiles;
  int l = 0;
  for (int j = 1; j < a.n; ++j)
    if (t >= a.layer[j].first) l = j;
  const Layer& y = a.layer[l];
  if constexpr (PLAIN) run_tile<false, false>(a, y, t - y.first, worker, lds);
  else if (y.ry) run_tile<true, true>(a, y, t - y.first, worker, lds);
  else run_tile<true, false>(a, y, t - y.first, worker, lds);
}

}  // namespace f32g

// Meant for models whose weight gradients last about as long as a launch: 64 x 64 tiles of all layers and workers, times the samples.
// Larger ones have the layers' own launches run beside the data gradients on the side stream.  Step of each, grouped / not:
// 512-512-512-10, 16 workers of 64 samples (139 thousand) 187 / 201 us, 3072-1024-512-10, four of 64 (231) 236 / 241, 512-512-512-10, eight of
// 256 or four of 512 (278) 207 / 197 and 201 / 191; first-order steps, four of 256 (139) 98 / 108, four of 512 (278) 142 / 142.
bool wgrad_group_f32_ok(const dw_config& c) {
  int64_t tiles = 0;
  for (int l = 1; l <= c.n_layers; ++l) tiles += (int64_t)((c.dims[l] + 63) / 64) * ((c.dims[l - 1] + 63) / 64);
  return tiles * c.k < 4096 && tiles * c.k * c.batch < 250000;
}

hipError_t launch_wgrad_group_f32(const GemmArgs* layers, int n, hipStream_t s) {
  KernelScope ks(KC_GEMM_WGRAD, s);
  f32g::Args a{};
  a.n = n; a.B = layers[0].K; a.Pp = layers[0].c_wstride; a.active_mask = layers[0].active_mask;
  a.workers = active_count(a.active_mask, layers[0].k);
  a.g = reinterpret_cast<float*>(layers[0].C); a.hz = reinterpret_cast<float*>(layers[0].RC);
  for (int j = 0; j < n; ++j) {
    const GemmArgs& in = layers[j];
    f32g::Layer& y = a.layer[j];
    y.x = reinterpret_cast<const float*>(in.X); y.rx = reinterpret_cast<const float*>(in.RX);
    y.y = reinterpret_cast<const float*>(in.Y); y.ry = reinterpret_cast<const float*>(in.RY);
    y.x_wstride = in.x_wstride; y.y_wstride = in.y_wstride;
    y.woff = reinterpret_cast<float*>(in.C) - a.g; y.boff = in.gb - a.g;         // (from the first layer's W)
    y.ldx = in.ldx; y.M = in.M; y.N = in.N; y.tiles_m = (in.M + f32g::EDGE - 1) / f32g::EDGE;
    y.first = a.tiles;
    a.tiles += y.tiles_m * ((in.N + f32g::EDGE - 1) / f32g::EDGE);
  }
  const dim3 grid = xcd_grid((int64_t)a.tiles * a.workers);
  const int smem = 3 * f32g::EDGE * kRowBytes * (layers[0].plain ? 2 : 4);       // 48 KB: three blocks to a compute unit
  if (layers[0].plain) hipLaunchKernelGGL(f32g::wgrad_group_f32<true>, grid, dim3(f32g::NT), smem, s, a);
  else hipLaunchKernelGGL(f32g::wgrad_group_f32<false>, grid, dim3(f32g::NT), smem, s, a);
  return hipGetLastError();
}

// c = the sum over the slices of p[slice * step], rc the same of p[slice * step + second], added in slice order.  One load at
// a time this is bound by the memory's latency, slice after slice, so eight slices' loads go out together (small CNN, ten
// workers, three weight gradients in tens of slices: 25 -> 9.4 us each; 15.3 with the loads of the bias sums still serial).
__device__ __forceinline__ void sum_slices(const float* p, int64_t step, int64_t second, int slices, bool plain, float& c, float& rc) {
  constexpr int kInFlight = 8;
  c = 0.f; rc = 0.f;
  int sl = 0;
  for (; sl + kInFlight <= slices; sl += kInFlight) {
    float v[kInFlight], rv[kInFlight];
#pragma unroll
    for (int j = 0; j < kInFlight; ++j) {
      v[j] = p[(sl + j) * step];
      rv[j] = plain ? 0.f : p[(sl + j) * step + second];
    }
#pragma unroll
    for (int j = 0; j < kInFlight; ++j) { c += v[j]; rc += rv[j]; }
  }
  for (; sl < slices; ++sl) {
    c += p[sl * step];
    if (!plain) rc += p[sl * step + second];
  }
}

// adds the slices of a product cut along its contraction, in slice order, and applies the epilogue the main kernel
// left out: C, RC (M rows of ldc, columns < N) and, for a weight gradient, the bias sums gb, hzb (M)
__global__ __launch_bounds__(256) void sum_slices_kernel(GemmArgs a) {
  const int worker = nth_active_worker(a.active_mask, blockIdx.y);
  const int64_t n_out = (int64_t)a.M * a.ldc;
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int n = (int)(e % a.ldc);
  if (e < n_out && n < a.N) {
    float c, rc;
    sum_slices(a.part + (int64_t)worker * 2 * a.part_stride + e, (int64_t)a.k * 2 * a.part_stride, a.part_stride, a.ksplit,
               a.plain != 0, c, rc);
    if (a.epi == EPI_RELU) {
      const uint32_t* zb = a.zbits + (int64_t)worker * a.z_stride;
      const int64_t bi = a.zb_off + n;
      c += a.bias[(int64_t)worker * a.bias_wstride + n];
      if (!a.plain) rc += ((zb[bi >> 5] >> (bi & 31)) & 1u) ? 1.f : -1.f;
      if (!(c > 0.f)) { c = 0.f; rc = 0.f; }
    } else if (a.epi == EPI_MASK) {
      const float* msk = reinterpret_cast<const float*>(a.mask_src) + (int64_t)worker * a.mask_wstride;
      if (!(msk[(e / a.ldc) * a.ld_mask + n] > 0.f)) { c = 0.f; rc = 0.f; }
    }
    reinterpret_cast<float*>(a.C)[(int64_t)worker * a.c_wstride + e] = c;
    if (!a.plain) reinterpret_cast<float*>(a.RC)[(int64_t)worker * a.c_wstride + e] = rc;
  }
  if (a.epi == EPI_WGRAD && e < a.M) {
    float b, rb;
    sum_slices(a.part_b + (int64_t)worker * 2 * a.M + e, (int64_t)a.k * 2 * a.M, a.M, a.ksplit, a.plain != 0, b, rb);
    a.gb[(int64_t)worker * a.c_wstride + e] = b;
    if (!a.plain) a.hzb[(int64_t)worker * a.c_wstride + e] = rb;
  }
}

// a kernel instance with its dynamic LDS
template <int BM, int BN, int WM, int WN, bool X_KC, bool Y_KC, bool HAS_RX, int RYM, int EPI, int FM = 0, int XV = VIEW_NONE,
          int YV = VIEW_NONE>
static hipError_t launch_instance(const GemmArgs& a, dim3 grid, hipStream_t s) {
  constexpr int smem = gemm_f32_lds(BM, BN, WM, WN, HAS_RX, RYM, EPI);
  static_assert(smem <= 160 * 1024 - 256, "a compute unit's LDS");
  auto kern = dual_gemm_f32<BM, BN, WM, WN, X_KC, Y_KC, HAS_RX, RYM, EPI, FM, XV, YV>;
  if (smem > 64 * 1024) {
    static LdsLimitOnce lim;
    const hipError_t e = lim.raise(reinterpret_cast<const void*>(kern), smem);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, grid, dim3(WM * WN * 64), smem, s, a);
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN>
static hipError_t launch_shape(const GemmArgs& a, hipStream_t s) {
  const int64_t tiles = (int64_t)((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  const bool sliced = a.ksplit > 1;
  const int workers = active_count(a.active_mask, a.k);
  const dim3 grid = xcd_grid(tiles * (sliced ? a.ksplit : 1) * workers);
  const bool rx = a.RX != nullptr;
  hipError_t e;
#define DW_GO(...) e = launch_instance<BM, BN, WM, WN, __VA_ARGS__>(a, grid, s)
  if (a.x_view != VIEW_NONE || a.y_view != VIEW_NONE) {
    // a convolution on a map: forward (patches as X), weight gradient (patches as Y), data gradient (the gradient
    // map seen from the input positions as X, the taps of W in the contraction index)
    if (a.epi == EPI_RELU && rx && a.x_view == VIEW_PATCH && a.y_view == VIEW_NONE)
      DW_GO(true, true, true, RY_BITS, EPI_RELU, 0, VIEW_PATCH, VIEW_NONE);
    else if (a.epi == EPI_WGRAD && a.RY && a.x_view == VIEW_NONE && a.y_view == VIEW_PATCH)
      DW_GO(false, false, true, RY_MEM, EPI_WGRAD, 0, VIEW_NONE, VIEW_PATCH);
    else if (a.epi == EPI_MASK && a.x_view == VIEW_SHIFTED && a.y_view == VIEW_TAPS)
      DW_GO(true, false, true, RY_BITS, EPI_MASK, 0, VIEW_SHIFTED, VIEW_TAPS);
    else
      return hipErrorInvalidValue;
  } else if (a.plain) {
    // a first-order step: the plain products alone
    if (a.epi == EPI_RELU) DW_GO(true, true, false, RY_NONE, EPI_RELU);
    else if (a.epi == EPI_MASK) DW_GO(true, false, false, RY_NONE, EPI_MASK);
    else if (a.epi == EPI_WGRAD) DW_GO(false, false, false, RY_NONE, EPI_WGRAD);
    else return hipErrorInvalidValue;
  } else if (a.r_only && !sliced && a.epi == EPI_RELU) {
    // a later Hutchinson probe of the same minibatch: the plain product is in memory, only the R-products are computed
    if (rx) DW_GO(true, true, true, RY_BITS, EPI_RELU, 1); else DW_GO(true, true, false, RY_BITS, EPI_RELU, 1);
  } else if (a.r_only && !sliced && a.epi == EPI_MASK) {
    DW_GO(true, false, true, RY_BITS, EPI_MASK, 1);
  } else if (a.epi == EPI_RELU) {              // forward, hidden layer
    if (rx) DW_GO(true, true, true, RY_BITS, EPI_RELU); else DW_GO(true, true, false, RY_BITS, EPI_RELU);
  } else if (a.epi == EPI_MASK) {              // data gradient
    DW_GO(true, false, true, RY_BITS, EPI_MASK);
  } else if (a.epi == EPI_WGRAD) {             // weight gradient
    if (a.RY) DW_GO(false, false, true, RY_MEM, EPI_WGRAD); else DW_GO(false, false, true, RY_NONE, EPI_WGRAD);
  } else {
    return hipErrorInvalidValue;
  }
#undef DW_GO
  if (e != hipSuccess) return e;
  if (sliced) {
    const int64_t n_out = (int64_t)a.M * a.ldc;
    hipLaunchKernelGGL(sum_slices_kernel, dim3((unsigned)((n_out + 255) / 256), (unsigned)workers), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

// Weight gradient that applies the update itself: 64 x 128 tiles, four waves of 32 x 64, so that two blocks share a compute
// unit (74 KB of LDS, 256 registers) and one's update traffic runs under the other's products.
constexpr int kFuseBM = 64, kFuseBN = 128;
template <int FM>
static hipError_t launch_fused_wgrad_mode(const GemmArgs& a, hipStream_t s) {
  const dim3 grid = xcd_grid((int64_t)(a.M / kFuseBM) * (a.N / kFuseBN) * active_count(a.active_mask, a.k));
  if (a.RY) return launch_instance<kFuseBM, kFuseBN, 2, 2, false, false, true, RY_MEM, EPI_WGRAD_FUSED, FM>(a, grid, s);
  return launch_instance<kFuseBM, kFuseBN, 2, 2, false, false, true, RY_NONE, EPI_WGRAD_FUSED, FM>(a, grid, s);
}

// several Hutchinson probes: own instances for the probes before the last and for the last one
static hipError_t launch_fused_wgrad(const GemmArgs& a, hipStream_t s) {
  if (a.fu.probe_mode == 1) return launch_fused_wgrad_mode<1>(a, s);
  if (a.fu.probe_mode == 2) return launch_fused_wgrad_mode<2>(a, s);
  return launch_fused_wgrad_mode<0>(a, s);
}

// The fp32 weight-gradient product of W[n_out][n_in] can apply the update in its epilogue when W is made of whole
// 128 x 128 tiles that fill the chip, an averaging block is at most 32 and the Hessian power is 1.
bool gemm_f32_wgrad_fusable(int n_out, int n_in, int k, int avg_block, float hpow, int64_t woff) {
  if (n_out % 128 != 0 || n_in % 128 != 0 || woff % 32 != 0 || avg_block > 32 || hpow != 1.0f) return false;
  if ((int64_t)n_out * n_in >= (1ll << 31)) return false;
  return (int64_t)(n_out / 128) * (n_in / 128) * k >= 512;
}
int gemm_f32_wgrad_tiles(int n_out, int n_in) { return (n_out / 128) * (n_in / 128); }   // partial-sum slots

hipError_t launch_gemm_f32(const GemmArgs& a, hipStream_t s) {
  KernelScope ks(a.epi == EPI_WGRAD ? KC_GEMM_WGRAD : a.epi == EPI_MASK ? KC_GEMM_DGRAD : KC_GEMM_FWD, s);
  if (a.epi == EPI_WGRAD && a.fu.on) return launch_fused_wgrad(a, s);
  if (a.N <= 32) return launch_shape<128, 32, 4, 1>(a, s);
  if (a.M <= 32) return launch_shape<32, 128, 1, 4>(a, s);
  if (a.N <= 64 && (int64_t)((a.M + 127) / 128) * a.k >= 512) return launch_shape<128, 64, 4, 1>(a, s);   // many rows, few columns
  return launch_shape<64, 64, 2, 2>(a, s);
}

}  // namespace dw
