// One worker step of a small fp32 MLP in a single kernel (gfx950, wave64).
//
// A model whose parameters and activations fit in the LDS of one compute unit spends its step waiting for a chain of
// short kernels (Rademacher bits, a product and its sum of slices per layer and direction, head, update: 9 launches of
// 2 to 7 us each for a 32-64-10 model).  Here one block per worker keeps everything on chip and walks through the
// whole of Section IV-B: z from the counter-based stream, forward and R-forward pass, softmax head, backward and
// R-backward pass (g and the Hessian-vector product Hz, Section II eq.(2) and the Hutchinson display), D = z*Hz with
// its block mean along fan-in, moments, bias correction, parameter update (eq.(4)) and the squared distance of the
// new parameters to the centre for the next communication round (Section V-B).
//
// What bounds it is the chain of phases between barriers, each a trip through LDS and some hundred instructions of one wave, so
// every phase spreads tiles over the waves and has few instructions a wave.  The products are 16 x 16 tiles on the fp32 matrix
// instruction, a wave each, in several chains added at the end (TileSums): forward products and data gradients four, weight gradients and
// contractions of up to 16 two; four k of an operand come with one LDS read.  A thread owns up to four groups of four consecutive parameters: it loads a group, draws its four signs from the stream
// (no sign words pass through LDS), puts both into LDS and applies the group's update at the end; the loads of the update go
// out with the first ones.  Barriers wait for LDS alone.  32-64-10, four workers of 16 samples: kernel 20.7 -> 12.2 us, 2 of them
// until the first loads are there (products as multiply-add loops, one output per thread with 4-byte reads and one sample per thread in
// the head: 20.7; four samples a thread, 16-byte reads and 16 lanes per sample: 12.4).
//
// LDS (floats): W_l with rows of an odd number of 16-byte units (so that lanes that own consecutive rows j read different
// banks), b_l, the same layout for z as +-1 floats, a_0, then a_l and Ra_l of the hidden layers, two pairs of error buffers
// (d_l, Rd_l and d_{l-1}, Rd_{l-1}), and g, Hz in the canonical layout (the first layer's in place of its W and z).
#include <cstddef>
#include <type_traits>

#include "dw_internal.h"
#include "dw_device_util.h"
#include "dw_head_math.h"

namespace dw {

namespace {

constexpr int kTinyThreads = 1024;                  // 16 waves on the one compute unit: four per SIMD hide the LDS latency
constexpr int kTinyWaves = kTinyThreads / 64;
constexpr int kTinyMaxLdsFloats = 40 * 1024 - 128;  // the compute unit's 160 KB but for what the kernel declares itself

constexpr int kTinyGroups = 4;                      // groups of four parameters a thread may own

struct TinyLayer {
  int woff;                                          // canonical offset of W_l (its bias follows)
  int pos, ws;                                       // LDS offset of W_l's padded rows and their length (the bias follows the rows)
  uint32_t by_q, by_tiles_k;                         // multipliers of the divisions by d_{l-1} / 4 and its number of tiles (see divide)
};

struct TinyArgs {
  const float* x; const int32_t* y;                  // [k][B][d_0], [k][B]
  const uint32_t* zbits_in; int64_t z_stride_in;     // caller's sign bits, or nullptr: drawn here
  uint32_t* zbits; int64_t z_stride;                 // the library's sign-bit buffer (written when drawn here)
  float* theta; float* m; float* v; float* g; float* hz; const float* centre;
  double* partials; int n_blocks;                    // [k][n_blocks] squared-distance partial sums
  float* act[DW_MAX_LAYERS];                         // a_l of the hidden layers in memory, [k][B][d_l] (index l)
  float* loss;                                       // [k] or nullptr
  int64_t P, Pp;
  int L, B, k;
  int dims[DW_MAX_LAYERS + 1];
  TinyLayer layer[DW_MAX_LAYERS];                    // index l-1
  int wsize, hidden, dmax;                           // floats of the padded parameters; sum of the hidden widths; row length of the errors
  uint32_t by_tiles_m;                               // of the division by the tiles of the minibatch
  int avg_block;
  float lr, beta1, beta2, eps, hpow;
  uint64_t active_mask;
  uint64_t key[DW_MAX_K];                            // keys of the workers' Rademacher streams at this step
  UpdateScalars sc;
};

__device__ __forceinline__ uint64_t tiny_mix64(uint64_t x) {     // SplitMix64 output function
  x ^= x >> 30; x *= 0xBF58476D1CE4E5B9ull;
  x ^= x >> 27; x *= 0x94D049BB133111EBull;
  x ^= x >> 31;
  return x;
}

__device__ __forceinline__ float tiny_denom(float vhat, float hpow) {       // (sqrt(v_hat))^hpow
  if (hpow == 1.0f) return sqrtf(vhat);
  if (hpow == 0.0f) return 1.0f;
  if (hpow == 2.0f) return vhat;
  return powf(vhat, 0.5f * hpow);
}

// x / d for x < 2^16 with by = floor(2^32 / d) + 1 (0 for d = 1)
__host__ inline uint32_t divisor(int d) { return d == 1 ? 0u : (uint32_t)((1ull << 32) / (uint64_t)d + 1); }
__device__ __forceinline__ int divide(int x, uint32_t by) { return by == 0u ? x : (int)__umulhi((uint32_t)x, by); }

__device__ __forceinline__ const float4& at4(const float* p) { return *reinterpret_cast<const float4*>(p); }

// Everything the threads of the block tell each other goes through LDS, so a barrier need not wait for stores to memory
// (__syncthreads does: up to 2 us of a step)
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

typedef float f4 __attribute__((ext_vector_type(4)));
constexpr f4 kZero4 = {0.f, 0.f, 0.f, 0.f};
__device__ __forceinline__ f4 mfma(float x, float y, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, c, 0, 0, 0); }

// A 16 x 16 tile of C = X*Y, RC = RX*Y + X*V.  Several chains of accumulation, added at the end: the matrix instruction's sums are
// further from the exact ones than a chain of multiply-adds of the same length, several of a quarter or half of it are closer.  Relative
// error of g and Hz, worst layer, here / as multiply-add loops: 32-64-10 with 16 samples 10e-8 / 14e-8, with 64 12e-8 / 18e-8; 64-14
// with 256 21e-8 / 29e-8; 8-8-3 with 400 20e-8 / 28e-8.
template <int CHAINS>
struct TileSums {
  f4 c[CHAINS], xv[CHAINS], ry[CHAINS];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int h = 0; h < CHAINS; ++h) c[h] = xv[h] = ry[h] = kZero4;
  }
  // sixteen k, four with each lane (chains h and h + 1)
  __device__ __forceinline__ void sixteen(int h, const f4& x, const f4& y, const f4& v, bool has_rx, const f4& rx) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      c[h + (j & 1)] = mfma(x[j], y[j], c[h + (j & 1)]);
      xv[h + (j & 1)] = mfma(x[j], v[j], xv[h + (j & 1)]);
    }
    if (has_rx) {
#pragma unroll
      for (int j = 0; j < 4; ++j) ry[h + (j & 1)] = mfma(rx[j], y[j], ry[h + (j & 1)]);
    }
  }
  __device__ __forceinline__ f4 plain() const { return CHAINS == 4 ? (c[0] + c[1]) + (c[2] + c[CHAINS - 1]) : c[0] + c[1]; }
  __device__ __forceinline__ f4 companion() const {
    return CHAINS == 4 ? ((xv[0] + xv[1]) + (xv[2] + xv[CHAINS - 1])) + ((ry[0] + ry[1]) + (ry[2] + ry[CHAINS - 1]))
                       : (xv[0] + xv[1]) + (ry[0] + ry[1]);
  }
};

// the tile of rows a (16 samples' rows, this lane's one) and w, z (16 outputs' rows, this lane's one), kg: the lane's four of 16 k
__device__ __forceinline__ void forward_tile(TileSums<4>& t, const float* a, const float* ra, const float* w, const float* z, int kg, int din) {
  t.clear();
  for (int k0 = 0; k0 < din; k0 += 32) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = k0 + 16 * h + 4 * kg;
      f4 x = kZero4, rx = kZero4, y = kZero4, v = kZero4;
      if (k < din) {
        x = *reinterpret_cast<const f4*>(a + k); y = *reinterpret_cast<const f4*>(w + k); v = *reinterpret_cast<const f4*>(z + k);
        if (ra) rx = *reinterpret_cast<const f4*>(ra + k);
      }
      if (k0 + 16 * h < din) t.sixteen(2 * h, x, y, v, ra != nullptr, rx);       // (uniform)
    }
  }
}

// GP: groups of four parameters per thread
template <int GP>
__global__ __launch_bounds__(kTinyThreads) void tiny_step_kernel(TinyArgs a) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = blockIdx.x;                                    // one block per worker
  const bool active = (a.active_mask >> i) & 1ull;
  const int L = a.L, B = a.B;
  const int P = (int)a.P;
  __shared__ double red[kTinyThreads / 64];
  float nsum = 0.f;
  float* th_g = a.theta + (int64_t)i * a.Pp;

  if (active) {
    // per-worker scalars from the kernel-argument block (scalar loads; indexing the by-value argument with a
    // variable would copy it to scratch memory)
    typedef const char __attribute__((address_space(4)))* karg_bytes;
    typedef const float __attribute__((address_space(4)))* karg_floats;
    typedef const uint64_t __attribute__((address_space(4)))* karg_u64;
    const karg_bytes ka = (karg_bytes)__builtin_amdgcn_kernarg_segment_ptr();
    const uint64_t key = ((karg_u64)(ka + offsetof(TinyArgs, key)))[i];
    const karg_floats bc = (karg_floats)(ka + offsetof(TinyArgs, sc));
    const float ib1 = bc[i], ib2 = bc[DW_MAX_K + i];
    static_assert(offsetof(UpdateScalars, inv_bc2) == DW_MAX_K * sizeof(float), "inv_bc2 follows inv_bc1");

    float* Wp = lds;                                           // padded weights and biases, layer after layer
    float* Zp = Wp + a.wsize;                                  // z as +-1 in the same layout
    float* A0 = Zp + a.wsize;                                  // a_0 [B][d_0]
    float* AH = A0 + B * a.dims[0];                            // a_l, Ra_l of the hidden layers, [B][d_l] each
    const int dmax = a.dmax;
    float* DB = AH + 2 * B * a.hidden;                         // error buffers: 2 x (d, Rd), [B][dmax] each
    float* LV = DB + 4 * B * dmax;                             // per sample what its loss is made of, [2][B]
    // g and Hz in the canonical layout: the first layer's where its parameters were (read only by its forward product), the others'
    const int P1 = a.dims[1] * (a.dims[0] + 1);
    float* GL = LV + ((2 * B + 3) & ~3); float* HL = GL + (((P - P1) + 3) & ~3);
    const int r16 = lane & 15, kg = lane >> 4;                 // place in a 16 x 16 tile's operands

    // ---- this thread's parameters, the input minibatch, the signs ---------------------------------------------
    const int nq = (P + 3) >> 2;
    float4 T0 = make_float4(0.f, 0.f, 0.f, 0.f), M0 = T0, V0 = T0, C0 = T0;      // the first group's state, kept for the update
    float4 T[GP];
#pragma unroll
    for (int u = 0; u < GP; ++u) {
      const int q = u * kTinyThreads + tid;
      T[u] = q < nq ? at4(th_g + 4 * q) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (tid < nq) {
      T0 = T[0];
      M0 = at4(a.m + (int64_t)i * a.Pp + 4 * tid);
      V0 = at4(a.v + (int64_t)i * a.Pp + 4 * tid);
      C0 = at4(a.centre + 4 * tid);
    }
    const float* xs = a.x + (int64_t)i * B * a.dims[0];
    const int nx = B * a.dims[0] / 4;
    const float4 X0 = tid < nx ? at4(xs + 4 * tid) : make_float4(0.f, 0.f, 0.f, 0.f);
    const int n_first = 16 * (wave >> 2) + 4 * (lane >> 4) + (wave & 3);         // (see the output layer)
    const int y_first = n_first < B ? a.y[(int64_t)i * B + n_first] : 0;
    // where a group lies in Wp and in Zp (-1: nowhere), and whether it is of a bias
    bool is_bias[GP];
    uint32_t z4[GP];
    int g_at[GP];
#pragma unroll
    for (int u = 0; u < GP; ++u) {
      const int q = u * kTinyThreads + tid, e0 = q << 2;
      is_bias[u] = false; z4[u] = 0; g_at[u] = -1;
      if (q >= nq) continue;
      // element j of z: bit j % 64 of word j / 64 of the worker's stream, or the caller's
      if (a.zbits_in) {
        z4[u] = a.zbits_in[(int64_t)i * a.z_stride_in + (e0 >> 5)] >> (e0 & 31);
      } else {
        const uint64_t xw = tiny_mix64(key + 0x9E3779B97F4A7C15ull * (uint64_t)((e0 >> 6) + 1));
        if ((q & 15) == 0)
          reinterpret_cast<uint2*>(a.zbits + (int64_t)i * a.z_stride)[q >> 4] = make_uint2((uint32_t)xw, (uint32_t)(xw >> 32));
        z4[u] = (uint32_t)(xw >> (e0 & 63));
      }
      for (int l = 1; l <= L; ++l) {
        const TinyLayer& y = a.layer[l - 1];
        const int dout = a.dims[l], din = a.dims[l - 1], r = e0 - y.woff, nw = dout * din;
        if (r < 0 || r >= nw + dout) continue;
        const int row = r < nw ? divide(r >> 2, y.by_q) : dout;         // (the bias follows the last row)
        is_bias[u] = r >= nw;
        g_at[u] = y.pos + row * y.ws + (r - (is_bias[u] ? nw : row * din));
      }
      *reinterpret_cast<float4*>(Zp + g_at[u]) = make_float4((z4[u] & 1u) ? 1.f : -1.f, (z4[u] & 2u) ? 1.f : -1.f,
                                                             (z4[u] & 4u) ? 1.f : -1.f, (z4[u] & 8u) ? 1.f : -1.f);
    }
    // (what was loaded is looked at only now)
#pragma unroll
    for (int u = 0; u < GP; ++u)
      if (g_at[u] >= 0) *reinterpret_cast<float4*>(Wp + g_at[u]) = T[u];
    if (tid < nx) reinterpret_cast<float4*>(A0)[tid] = X0;
    for (int e = tid + kTinyThreads; e < nx; e += kTinyThreads) reinterpret_cast<float4*>(A0)[e] = at4(xs + 4 * e);
    lds_barrier();

    // ---- hidden layers, forward and R-forward: s = a W^T + b, Rs = Ra W^T + a V^T + c; a wave per tile ------------
    const int tiles_m = (B + 15) >> 4;
    const float* Ain = A0; const float* RAin = nullptr;
    float* hid = AH;
    for (int l = 1; l < L; ++l) {
      const TinyLayer& y = a.layer[l - 1];
      const int dout = a.dims[l], din = a.dims[l - 1], ws = y.ws;
      float* Aout = hid; float* RAout = hid + B * dout;
      float* act_g = a.act[l] + (int64_t)i * B * dout;
      for (int tile = wave; tile < tiles_m * ((dout + 15) >> 4); tile += kTinyWaves) {
        const int tn = divide(tile, a.by_tiles_m), m0 = (tile - tn * tiles_m) << 4, n = 16 * tn + r16;
        // rows past the end repeat the last one (not stored)
        const int m = m0 + r16 < B ? m0 + r16 : B - 1, j = n < dout ? n : dout - 1;
        TileSums<4> t;
        forward_tile(t, Ain + m * din, RAin ? RAin + m * din : nullptr, Wp + y.pos + j * ws, Zp + y.pos + j * ws, kg, din);
        const float b = Wp[y.pos + dout * ws + j], c = Zp[y.pos + dout * ws + j];
        const f4 s = t.plain(), rs = t.companion();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = m0 + 4 * kg + r, at = row * dout + n;
          const float v = s[r] + b, rv = rs[r] + c;
          const bool on = v > 0.f;                             // ReLU: slope 0 at exactly 0
          if (row < B && n < dout) { Aout[at] = on ? v : 0.f; RAout[at] = on ? rv : 0.f; act_g[at] = on ? v : 0.f; }
        }
      }
      lds_barrier();
      Ain = Aout; RAin = RAout; hid += 2 * B * dout;
    }

    // ---- output layer and softmax cross-entropy head: d_L = (p - onehot)/B, Rd_L.  A row of 16 lanes holds the logits of four
    // samples, one class a lane; four waves compute the same tile and each goes on with one of the four ------------
    float* Dl = DB; float* RDl = DB + B * dmax;                // errors of layer l
    float* Dn = DB + 2 * B * dmax; float* RDn = DB + 3 * B * dmax;       // errors of layer l-1
    {
      const TinyLayer& y = a.layer[L - 1];
      const int C = a.dims[L], din = a.dims[L - 1], j = r16 < C ? r16 : C - 1;
      for (int unit = wave; unit < 4 * tiles_m; unit += kTinyWaves) {    // (uniform: all lanes take the moves)
        const int m0 = (unit >> 2) << 4, m = m0 + r16 < B ? m0 + r16 : B - 1, sample = m0 + 4 * kg + (unit & 3);
        const int label = unit == wave ? y_first : sample < B ? a.y[(int64_t)i * B + sample] : 0;
        TileSums<4> t;
        forward_tile(t, Ain + m * din, RAin ? RAin + m * din : nullptr, Wp + y.pos + j * y.ws, Zp + y.pos + j * y.ws, kg, din);
        const f4 s = t.plain(), rs = t.companion();
        const bool odd = unit & 1, up = unit & 2;
        const float sv = up ? (odd ? s[3] : s[2]) : (odd ? s[1] : s[0]), rv = up ? (odd ? rs[3] : rs[2]) : (odd ? rs[1] : rs[0]);
        float d, rd, rest, sy;
        head_lanes(sv + Wp[y.pos + C * y.ws + j], rv + Zp[y.pos + C * y.ws + j], r16, label, C, 1.0f / (float)B, d, rd, rest, sy);
        if (sample < B) {
          Dl[sample * dmax + r16] = d; RDl[sample * dmax + r16] = rd;
          if (r16 == 0) { LV[sample] = rest; LV[B + sample] = sy; }
        }
      }
    }
    lds_barrier();
    if (a.loss && wave == kTinyThreads / 64 - 1) {
      double t = 0.0;
      for (int n = lane; n < B; n += 64) t += (double)(log1pf(LV[n]) - LV[B + n]);
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) t += __shfl_xor(t, o);
      if (lane == 0) a.loss[i] = (float)(t / (double)B);
    }

    // ---- backward and R-backward: per layer the tiles of the data gradient and of the weight gradient and the bias gradients, a
    // wave each -------------------------------------------------------------------------------------------------
    for (int l = L; l >= 1; --l) {
      const TinyLayer& y = a.layer[l - 1];
      const int dout = a.dims[l], din = a.dims[l - 1], ws = y.ws;
      if (l > 1) { hid -= 2 * B * din; Ain = hid; RAin = hid + B * din; } else { Ain = A0; RAin = nullptr; }
      const int tiles_k = (din + 15) >> 4, tiles_j = (dout + 15) >> 4;
      const int nd = l > 1 ? tiles_m * tiles_k : 0, nw = tiles_j * tiles_k, nb = (dout + 63) >> 6;
      float* gl = l > 1 ? GL + (y.woff - P1) : Wp; float* hl = l > 1 ? HL + (y.woff - P1) : Zp;
      for (int unit = wave; unit < nd + nw + nb; unit += kTinyWaves) {
        if (unit < nd) {
          // through W_l, masked by the ReLU of layer l-1: d' = (d W) * [a > 0], Rd' = (Rd W + d V) * [a > 0]
          const int tn = divide(unit, a.by_tiles_m), m0 = (unit - tn * tiles_m) << 4, n = 16 * tn + r16;
          const int m = m0 + r16 < B ? m0 + r16 : B - 1, col = n < din ? n : din - 1;
          TileSums<4> t;
          t.clear();
          for (int j0 = 0; j0 < dout; j0 += 32) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const int j = j0 + 16 * h + 4 * kg;
              f4 d = kZero4, rd = kZero4, w, z;
              if (j < dout) { d = *reinterpret_cast<const f4*>(Dl + m * dmax + j); rd = *reinterpret_cast<const f4*>(RDl + m * dmax + j); }
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const int at = y.pos + (j + e < dout ? j + e : dout - 1) * ws + col;
                w[e] = j + e < dout ? Wp[at] : 0.f; z[e] = j + e < dout ? Zp[at] : 0.f;
              }
              if (j0 + 16 * h < dout) t.sixteen(2 * h, d, w, z, true, rd);       // (uniform)
            }
          }
          const f4 ds = t.plain(), rds = t.companion();
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = m0 + 4 * kg + r;
            if (row < B && n < din) {
              const bool on = Ain[row * din + n] > 0.f;
              Dn[row * dmax + n] = on ? ds[r] : 0.f; RDn[row * dmax + n] = on ? rds[r] : 0.f;
            }
          }
        } else if (unit < nd + nw) {
          // gW = d^T a, HzW = Rd^T a + d^T Ra (sums over the minibatch), transposed: a lane gets four of a row of W
          const int tile = unit - nd, tj = divide(tile, y.by_tiles_k), k0 = (tile - tj * tiles_k) << 4, j = 16 * tj + r16;
          const int k = k0 + r16 < din ? k0 + r16 : din - 1, jc = j < dout ? j : dout - 1;
          TileSums<2> t;
          t.clear();
          for (int n0 = 0; n0 < B; n0 += 16) {
            f4 x, rx = kZero4, d, rd;                          // samples n0 + kg, n0 + 4 + kg, ...
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int n = n0 + 4 * e + kg, nc = n < B ? n : B - 1;
              x[e] = Ain[nc * din + k]; d[e] = Dl[nc * dmax + jc]; rd[e] = RDl[nc * dmax + jc];
              if (RAin) rx[e] = RAin[nc * din + k];
              if (n >= B) { x[e] = 0.f; rx[e] = 0.f; d[e] = 0.f; rd[e] = 0.f; }
            }
            t.sixteen(0, x, d, rd, RAin != nullptr, rx);
          }
          const int at = j * din + k0 + 4 * kg;
          if (j < dout && k0 + 4 * kg < din) {
            *reinterpret_cast<f4*>(gl + at) = t.plain();
            *reinterpret_cast<f4*>(hl + at) = t.companion();
          }
        } else {
          // column sums of d and Rd (columns past the classes are zero: the last group's tail)
          const int j = ((unit - nd - nw) << 6) + lane;
          if (j < ((dout + 3) & ~3)) {
            float gs = 0.f, hs = 0.f;
#pragma unroll 8
            for (int n = 0; n < B; ++n) { gs += Dl[n * dmax + j]; hs += RDl[n * dmax + j]; }
            gl[dout * din + j] = gs; hl[dout * din + j] = hs;
          }
        }
      }
      lds_barrier();
      float* t0 = Dl; Dl = Dn; Dn = t0; t0 = RDl; RDl = RDn; RDn = t0;
    }

    // ---- D = z*Hz, block mean along fan-in, moments, update (same arithmetic as update_kernel) ----------------
    {
      float* m_g = a.m + (int64_t)i * a.Pp; float* v_g = a.v + (int64_t)i * a.Pp;
      float* g_g = a.g + (int64_t)i * a.Pp; float* hz_g = a.hz + (int64_t)i * a.Pp;
      const float inv_b = 1.0f / (float)a.avg_block;
      const int group_lanes = a.avg_block >> 2;
#pragma unroll
      for (int u = 0; u < GP; ++u) {
        if (u * kTinyThreads >= nq) break;                     // (uniform: every lane takes the shuffles)
        const int q = u * kTinyThreads + tid;
        const bool valid = q < nq;
        const int e0 = q << 2;
        float4 M = M0, V = V0, Cn = C0;
        float4 Tq = T0;
        if (u > 0) {
          Tq = M = V = Cn = make_float4(0.f, 0.f, 0.f, 0.f);
          if (valid) { Tq = at4(th_g + e0); M = at4(m_g + e0); V = at4(v_g + e0); Cn = at4(a.centre + e0); }
        }
        const bool avg = !is_bias[u] && a.avg_block > 1;       // biases are not averaged
        float4 G = make_float4(0.f, 0.f, 0.f, 0.f), H = G;
        if (valid) { G = at4(e0 < P1 ? Wp + e0 : GL + (e0 - P1)); H = at4(e0 < P1 ? Zp + e0 : HL + (e0 - P1)); }
        const float g[4] = {G.x, G.y, G.z, G.w}, hz[4] = {H.x, H.y, H.z, H.w};
        float th[4] = {Tq.x, Tq.y, Tq.z, Tq.w}, mm[4] = {M.x, M.y, M.z, M.w}, vv[4] = {V.x, V.y, V.z, V.w};
        const float cc[4] = {Cn.x, Cn.y, Cn.z, Cn.w};
        float D[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) D[e] = ((z4[u] >> e) & 1u) ? hz[e] : -hz[e];     // Hutchinson: z * Hz
        float Ds[4] = {D[0], D[1], D[2], D[3]};
        if (a.avg_block == 2) {
          const float p0 = 0.5f * (D[0] + D[1]), p1 = 0.5f * (D[2] + D[3]);
          if (avg) { Ds[0] = Ds[1] = p0; Ds[2] = Ds[3] = p1; }
        } else if (a.avg_block >= 4) {
          float s = (D[0] + D[1]) + (D[2] + D[3]);
          for (int o = 1; o < group_lanes; o <<= 1) s += __shfl_xor(s, o);
          s *= inv_b;
          if (avg) { Ds[0] = Ds[1] = Ds[2] = Ds[3] = s; }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          mm[e] = a.beta1 * mm[e] + (1.0f - a.beta1) * g[e];
          vv[e] = a.beta2 * vv[e] + (1.0f - a.beta2) * (Ds[e] * Ds[e]);
          const float mhat = mm[e] * ib1, vhat = vv[e] * ib2;
          th[e] = th[e] - a.lr * (mhat / (tiny_denom(vhat, a.hpow) + a.eps));
          const float d = th[e] - cc[e];
          if (valid && e0 + e < P) nsum += d * d;
        }
        if (valid) {
          // (a last group that reaches past P touches the row's padding, which holds zeros and stays zero: g = Hz = 0)
          *reinterpret_cast<float4*>(th_g + e0) = make_float4(th[0], th[1], th[2], th[3]);
          *reinterpret_cast<float4*>(m_g + e0) = make_float4(mm[0], mm[1], mm[2], mm[3]);
          *reinterpret_cast<float4*>(v_g + e0) = make_float4(vv[0], vv[1], vv[2], vv[3]);
          *reinterpret_cast<float4*>(g_g + e0) = G;
          *reinterpret_cast<float4*>(hz_g + e0) = H;
        }
      }
    }
  } else {
    // a frozen worker only reports its distance to the centre
    const int nq = (P + 3) >> 2;
    for (int q = tid; q < nq; q += kTinyThreads) {
      const float4 t = at4(th_g + 4 * q), c = at4(a.centre + 4 * q);
      const float d0 = t.x - c.x, d1 = t.y - c.y, d2 = t.z - c.z, d3 = t.w - c.w;
      nsum += (d0 * d0 + d1 * d1) + (d2 * d2 + d3 * d3);
    }
  }
  double ws = (double)nsum;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) ws += __shfl_xor(ws, o);
  if (lane == 0) red[wave] = ws;
  lds_barrier();
  if (wave == 0) {
    double t = red[lane & (kTinyThreads / 64 - 1)];
#pragma unroll
    for (int o = kTinyThreads / 128; o >= 1; o >>= 1) t += __shfl_xor(t, o);
    if (lane < a.n_blocks) a.partials[(int64_t)i * a.n_blocks + lane] = lane == 0 ? t : 0.0;    // (n_blocks is 16 at most)
  }
}

// rows of an odd number of 16-byte units
int tiny_row(int din) { return din % 8 == 4 ? din : din + 4; }

int tiny_lds_floats(const dw_config& c, const Layout& lay) {
  int64_t wsize = 0, hidden = 0, dmax = DW_MAX_CLASSES;
  for (int l = 1; l <= c.n_layers; ++l) {
    wsize += (int64_t)c.dims[l] * tiny_row(c.dims[l - 1]) + (c.dims[l] + 3) / 4 * 4;
    if (l < c.n_layers) { hidden += c.dims[l]; if (c.dims[l] > dmax) dmax = c.dims[l]; }
  }
  const int64_t B = c.batch;
  const int64_t total = 2 * wsize + B * c.dims[0] + 2 * B * hidden + 4 * B * dmax + 2 * B + 3 + 2 * ((lay.P - (int64_t)c.dims[1] * (c.dims[0] + 1) + 3) / 4 * 4);
  return total > (1 << 30) ? (1 << 30) : (int)total;
}

// What the step of a model this size touches, in floats: parameters and signs with rows of an odd length, the minibatch, activations and
// errors with their companions, g and Hz of all layers, the sign words
int64_t tiny_size(const dw_config& c, const Layout& lay) {
  int64_t rows = 0, hidden = 0, dmax = DW_MAX_CLASSES;
  for (int l = 1; l <= c.n_layers; ++l) {
    rows += (int64_t)c.dims[l] * (c.dims[l - 1] + 2);
    if (l < c.n_layers) { hidden += c.dims[l]; if (c.dims[l] > dmax) dmax = c.dims[l]; }
  }
  const int64_t B = c.batch;
  return 2 * rows + B * c.dims[0] + 2 * B * hidden + 4 * B * dmax + 2 * ((lay.P + 3) / 4 * 4) + 2 * ((lay.P + 63) / 64) + B + 64;
}

}  // namespace

// A model takes this path when it is fp32 without a convolutional front end, one Hutchinson probe per step, the
// AdaHessian step, an averaging block inside one wave's reach, four groups of four parameters for every thread, and its size at most
// kTinyMaxSize (it then fits in LDS, which the last line makes sure of).
// The kernel could hold models up to a third larger, since g and Hz of the first layer lie where its parameters were.  Those keep to the
// launches of a layer each, because the sums there, in bf16 pieces, are closer to the 64-bit ones than the fp32 instruction's.  Relative
// error of g and Hz, worst layer, here / there, and the step with a round: 64-96-16, one worker of 16 samples: 11.3e-8 / 7.8e-8, 22 / 35 us;
// 252-60-5, one of 8: 16.7e-8 / 8.9e-8, 20 / 33; 512-16-100-15, one of one: 25e-8 / 8.1e-8; without a hidden layer they are slower too
// (80-14, one of 256: 21e-8 / 12e-8, 37 / 31 us).  Smaller models gain more by the one launch (32-64-10, one of 64: 11.8e-8 / 7.9e-8,
// 23.5 / 34 us; one of 16: 14.8 / 33).
constexpr int64_t kTinyMaxSize = 39 * 1024;
bool tiny_step_ok(const dw_config& c, const Layout& lay) {
  if (c.n_layers < 1 || c.dtype != DW_F32 || c.n_conv != 0 || c.n_samples > 1 || c.optimizer != DW_OPT_ADAHESSIAN)
    return false;
  if (c.avg_block > 64 || lay.P > 4 * kTinyGroups * kTinyThreads || c.batch > 1024) return false;
  return tiny_size(c, lay) <= kTinyMaxSize && tiny_lds_floats(c, lay) <= kTinyMaxLdsFloats;
}

hipError_t launch_tiny_step(const dw_config& c, char* ws, const Layout& lay, const void* d_x, const int32_t* d_y,
                            const uint32_t* d_zbits, const UpdateArgs& u, const uint64_t* keys_host, float* d_loss,
                            hipStream_t s) {
  KernelScope ks(KC_STEP, s);
  TinyArgs a{};
  a.x = reinterpret_cast<const float*>(d_x); a.y = d_y;
  a.zbits_in = d_zbits; a.z_stride_in = 2 * ((lay.P + 63) / 64);
  a.zbits = reinterpret_cast<uint32_t*>(ws + lay.zbits); a.z_stride = lay.z_stride;
  a.theta = u.theta; a.m = u.m; a.v = u.v; a.centre = u.centre;
  a.g = reinterpret_cast<float*>(ws + lay.g); a.hz = reinterpret_cast<float*>(ws + lay.hz);
  a.partials = u.partials; a.n_blocks = (int)lay.n_upd_blocks;
  for (int l = 1; l < c.n_layers; ++l) a.act[l] = reinterpret_cast<float*>(ws + lay.act[l]);
  a.loss = d_loss;
  a.P = lay.P; a.Pp = lay.Pp; a.L = c.n_layers; a.B = c.batch; a.k = c.k;
  for (int l = 0; l <= c.n_layers; ++l) a.dims[l] = c.dims[l];
  a.wsize = 0; a.hidden = 0; a.dmax = DW_MAX_CLASSES;
  a.by_tiles_m = divisor((c.batch + 15) / 16);
  for (int l = 1; l <= c.n_layers; ++l) {
    TinyLayer& y = a.layer[l - 1];
    y.woff = (int)lay.woff[l - 1]; y.pos = a.wsize; y.ws = tiny_row(c.dims[l - 1]);
    y.by_q = divisor(c.dims[l - 1] / 4); y.by_tiles_k = divisor((c.dims[l - 1] + 15) / 16);
    a.wsize += c.dims[l] * y.ws + (c.dims[l] + 3) / 4 * 4;
    if (l < c.n_layers) { a.hidden += c.dims[l]; if (c.dims[l] > a.dmax) a.dmax = c.dims[l]; }
  }
  a.avg_block = c.avg_block;
  a.lr = c.lr; a.beta1 = c.beta1; a.beta2 = c.beta2; a.eps = c.eps; a.hpow = c.hpow;
  a.active_mask = u.active_mask;
  for (int i = 0; i < DW_MAX_K; ++i) a.key[i] = i < c.k ? keys_host[i] : 0;
  a.sc = u.sc;
  const int smem = tiny_lds_floats(c, lay) * (int)sizeof(float);
  auto launch = [&](auto gp) -> hipError_t {
    auto kern = tiny_step_kernel<decltype(gp)::value>;
    static LdsLimitOnce lds_limit;                             // (one per instance of the lambda's body)
    const hipError_t e = lds_limit.raise(reinterpret_cast<const void*>(kern), kTinyMaxLdsFloats * (int)sizeof(float));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)c.k), dim3(kTinyThreads), smem, s, a);
    return hipGetLastError();
  };
  return lay.P <= 4 * kTinyThreads ? launch(std::integral_constant<int, 1>{}) : launch(std::integral_constant<int, kTinyGroups>{});
}

}  // namespace dw
