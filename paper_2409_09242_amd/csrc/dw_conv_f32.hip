// 3x3 convolutions of the front end beyond the first one, forward and data gradient, with their R-companions (Section VI's model,
// Section IV-B): C = sum over the nine taps of the shifted map times the tap's W, RC the same of the companion map plus the map
// times V.  Products in three bf16 pieces (dw_f32_pieces.h).
//
// As a product on patches every entry of the map is split into its pieces once for each tap that reads it, and the splitting,
// not the matrix cores, sets the pace.  Here a block takes the rows of the map around its positions, 32 channels (a cache line) at a time,
// splits them once into a slab in LDS, and the nine taps read the slab at nine offsets: positions as rows, a tap and 16 channels as a
// k-step.  The weights are few: a small launch before writes their pieces and signs for every k-step the way the lanes
// of the matrix instruction hold them, and the waves read them from there (the caches) straight into registers, two k-steps ahead,
// so that no barrier is met between the taps.  A wave owns 32 positions by 32 outputs; a block of eight waves, one to a
// compute unit, 256 positions by 32 outputs or 128 by 64, and goes on to further positions: the map's entries for the next slab are on
// their way while this one is multiplied.
// The data gradient is the same convolution of the gradient map, with a border of two, the taps in reverse and W transposed.
// Eight workers, 64 maps of 26 x 26 x 32 <-> 24 x 24 x 64: forward 207 -> 166 us, data gradient 384 -> 187 (as products on patches / now; the matrix
// instructions alone are 71 and 83 at 2.2 GHz).  By clock readings a slab of 36 k-steps for the two waves of a SIMD takes 27 thousand
// cycles, 17.3 of them matrix instructions, 3 the splitting, 1.5 the barriers, 5 waits inside; a block's end another 5.  Blocks of four waves, two to a
// compute unit, 16 channels a slab: 164 and 226 (each line of the map fetched twice, and both blocks split at the same time).
#include "dw_internal.h"
#include "dw_f32_pieces.h"

namespace dw {

namespace convf {

constexpr int NT = 512, WAVES = NT / 64, CH = 32, KS = 16;  // channels of a slab, of a k-step
constexpr int kPitch = 6 * CH * 2 + 16;                      // bytes of a slab position: pieces of the map, of its companion; sixteen
                                                             // consecutive positions' units use different banks
constexpr int kMostEntries = 384, kUnits = kMostEntries * 8 / NT;      // positions of a slab (150 KB); units of eight channels of a thread
constexpr int kFragBytes = 4 * 64 * 16;                      // of a k-step and 32 outputs: three pieces and the signs, 16 bytes a lane
static_assert(kUnits <= 9, "a unit beside a tap");
constexpr int kBlocks = 256;                                 // compute units

// the weight of output n, tap t, channel c: W[n * sn + t * st + c * sc], t counted back from 8 with `flip`
struct Weights { int N, C, sn, st, sc, flip; };
__host__ __device__ inline int ksteps_of(int C) { return (C + KS - 1) / KS * 9; }
__host__ __device__ inline int tiles_of(int N) { return (N + 31) / 32; }

struct Args {
  const float* in; const float* rin; int64_t in_wstride;     // [B][Hi][Wi][C]
  float* out; float* rout; const float* mask; int64_t out_wstride;     // [B][Ho][Wo][N]
  const char* frags; int64_t frag_wstride;                   // bytes
  const float* w; int64_t w_wstride; Weights ws;             // (for results that are not finite)
  const float* bias; const uint32_t* zbits; int64_t z_stride, z_off, zb_off;
  int B, Hi, Wi, Ho, Wo, pad, blocks, k;                     // blocks of an image
  uint32_t by_wv;                                            // floor(2^32 / (Wo + 2)) + 1
  uint64_t active_mask;
};

// EPI: EPI_RELU (bias, ReLU) or EPI_MASK (the ReLU mask of the map below); WN: waves side by side along the outputs
template <int WN, int EPI>
__global__ __launch_bounds__(NT) void conv3x3_f32(Args a) {
  constexpr int PB = WAVES / WN * 32;                        // positions of a block
  extern __shared__ __attribute__((aligned(16))) char slab[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, lhalf = lane >> 5;
  const int wm = wave / WN, C = a.ws.C, npos = a.Ho * a.Wo, Wv = a.Wo + 2, steps = ksteps_of(C), slabs = (C + CH - 1) / CH;
  const int ntiles = tiles_of(a.ws.N), groups = (ntiles + WN - 1) / WN;
  // units: 128 or 256 positions of an image and a group of outputs.  An XCD works through consecutive ones
  const unsigned per_worker = (unsigned)a.B * a.blocks * groups, units = per_worker * active_count(a.active_mask, a.k);
  const unsigned per_xcd = (units + 7) / 8, xcd = blockIdx.x & 7u, stride = gridDim.x >> 3;
  const unsigned end = (xcd + 1) * per_xcd < units ? (xcd + 1) * per_xcd : units;

  struct Unit { int worker, img, p0, y0, entries, group; };  // the slab: rows y0 .. of the map with its border, `entries` positions
  auto place = [&](unsigned u) {
    Unit r;
    const unsigned slot = u / per_worker, in_worker = u - slot * per_worker, block = in_worker / groups;
    r.worker = nth_active_worker(a.active_mask, slot);
    r.group = in_worker - block * groups;
    r.img = block / a.blocks; r.p0 = (block - r.img * a.blocks) * PB;
    r.y0 = r.p0 / a.Wo;
    const int y1 = ((r.p0 + PB < npos ? r.p0 + PB : npos) - 1) / a.Wo;
    r.entries = (y1 - r.y0 + 3) * Wv;
    return r;
  };
  // a thread's eight channels of every 64th position: of the map (threads 0 .. 3 of eight) or of its companion
  const int q = tid & 3, comp = (tid >> 2) & 1, e0 = tid >> 3;
  float4 raw[kUnits][2];
  unsigned inside = 0;                                       // bit b: unit b lies inside the map
  auto fetch = [&](const Unit& r, int s, int b) {            // one unit of the slab's
    const int e = e0 + b * 64, c = s * CH + q * 8;
    if (e >= r.entries) return;
    const float* src = (comp ? a.rin : a.in) + r.worker * a.in_wstride + (int64_t)r.img * a.Hi * a.Wi * C;
    const int vy = (int)__umulhi((uint32_t)e, a.by_wv), y = r.y0 + vy - a.pad, x = e - vy * Wv - a.pad;
    const bool ok = y >= 0 && y < a.Hi && x >= 0 && x < a.Wi;
    const float* p = src + (ok ? (y * a.Wi + x) * C : 0);
    inside = (inside & ~(1u << b)) | (ok ? 1u : 0u) << b;
    raw[b][0] = *reinterpret_cast<const float4*>(p + (c < C ? c : 0));
    raw[b][1] = *reinterpret_cast<const float4*>(p + (c + 4 < C ? c + 4 : 0));
  };
  auto store = [&](const Unit& r, int s) {
    const int c = s * CH + q * 8;
#pragma unroll
    for (int b = 0; b < kUnits; ++b) {
      const int e = e0 + b * 64;
      if (e >= r.entries) break;
      const bool k0 = (inside >> b & 1u) && c < C, k1 = (inside >> b & 1u) && c + 4 < C;
      const float f[8] = {k0 ? raw[b][0].x : 0.f, k0 ? raw[b][0].y : 0.f, k0 ? raw[b][0].z : 0.f, k0 ? raw[b][0].w : 0.f,
                          k1 ? raw[b][1].x : 0.f, k1 ? raw[b][1].y : 0.f, k1 ? raw[b][1].z : 0.f, k1 ? raw[b][1].w : 0.f};
      uint32_t o[3][4];
      split_pairs<false, 4>(f, o);
      char* to = slab + e * kPitch + comp * (3 * CH * 2) + q * 16;
#pragma unroll
      for (int j = 0; j < 3; ++j) *reinterpret_cast<uint4*>(to + j * CH * 2) = make_uint4(o[j][0], o[j][1], o[j][2], o[j][3]);
    }
  };
  // the weights' k-steps one after the other, unit after unit
  auto weights_of = [&](const Unit& r) {
    const int t = r.group * WN + wave % WN;
    return a.frags + r.worker * a.frag_wstride + (int64_t)(t < ntiles ? t : ntiles - 1) * steps * kFragBytes + lane * 16;
  };
  struct Frag { bf16x8 w[3], v; };
  const char* at_w; const char* next_w;
  int left;
  auto load = [&](Frag& f) {
#pragma unroll
    for (int c = 0; c < 3; ++c) f.w[c] = *reinterpret_cast<const bf16x8*>(at_w + c * 1024);
    f.v = *reinterpret_cast<const bf16x8*>(at_w + 3 * 1024);
    at_w += kFragBytes;
    if (--left == 0) { at_w = next_w; left = steps; }
  };

  unsigned u = xcd * per_xcd + (blockIdx.x >> 3);
  if (u >= end) return;
  Unit cur = place(u);
  Unit next = u + stride < end ? place(u + stride) : cur;
  at_w = weights_of(cur); next_w = weights_of(next); left = steps;
  Frag f0, f1;
  load(f0); load(f1);
#pragma unroll
  for (int b = 0; b < kUnits; ++b) fetch(cur, 0, b);
  const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (;;) {
    const int p = cur.p0 + wm * 32 + l32, pc = p < npos ? p : npos - 1;      // this lane's position (past the end: the last one, never stored)
    const int py = pc / a.Wo, px = pc - py * a.Wo;
    const char* at = slab + ((py - cur.y0) * Wv + px) * kPitch + lhalf * 16;
    const uint32_t* zb = a.zbits + cur.worker * a.z_stride;
    const int n = (cur.group * WN + wave % WN) * 32 + l32, nc = n < a.ws.N ? n : a.ws.N - 1;
    const int64_t o0 = cur.worker * a.out_wstride + (int64_t)cur.img * npos * a.ws.N + nc;
    floatx16 acc = zero, racc = zero, t = zero, tr = zero, sum = zero, rsum = zero;
    for (int s = 0; s < slabs; ++s) {
      __syncthreads();                                       // (everybody is done with the last slab)
      store(cur, s);
      __syncthreads();
      // the next slab's entries, a unit beside each of the first taps (a wave's loads arrive in order, and all at once they would
      // hold up the weights behind them)
      const bool same = s + 1 < slabs, more = same || u + stride < end;
      const Unit& ahead = same ? cur : next;
      const int ahead_s = same ? s + 1 : 0;
      for (int h = 0; h < 2 && s * CH + h * KS < C; ++h) {
        const char* from = at + h * KS * 2;
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
          Frag& f = tap & 1 ? f1 : f0;
          const char* row = from + ((tap / 3) * Wv + tap % 3) * kPitch;
          bf16x8 x[3], rx[3];
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            x[c] = *reinterpret_cast<const bf16x8*>(row + c * CH * 2);
            rx[c] = *reinterpret_cast<const bf16x8*>(row + (3 + c) * CH * 2);
          }
          if (tap < kUnits && h == 0 && more) fetch(ahead, ahead_s, tap);
          mfma6(x, f.w, acc, t);
          mfma6(rx, f.w, racc, tr);
          mfma3(x, f.v, racc, tr);
          load(f);
          __builtin_amdgcn_sched_barrier(0);                 // (taps pulled together spill)
        }
        const Frag swap = f0; f0 = f1; f1 = swap;            // (an odd number of taps)
        sum += acc; rsum += racc; acc = zero; racc = zero;   // (chains of nine: the instruction cuts sums off, an addition rounds)
      }
    }
    acc = sum; racc = rsum;
    bool finite = join_chains(acc, t);
    finite &= join_chains(racc, tr);
    if (__any(!finite)) {
      // a result that is not finite: the wave's tile again from whole numbers on the fp32 instruction (see dw_f32_pieces.h)
      const float* in = a.in + cur.worker * a.in_wstride + (int64_t)cur.img * a.Hi * a.Wi * C;
      const float* rin = a.rin + cur.worker * a.in_wstride + (int64_t)cur.img * a.Hi * a.Wi * C;
      const float* w = a.w + cur.worker * a.w_wstride;
      acc = zero; racc = zero;
      for (int tap = 0; tap < 9; ++tap)
        for (int c = lhalf; c < C; c += 2) {
          const int64_t o = (int64_t)nc * a.ws.sn + (a.ws.flip ? 8 - tap : tap) * a.ws.st + (int64_t)c * a.ws.sc, b = a.z_off + o;
          const float wv = w[o], vv = ((zb[b >> 5] >> (b & 31)) & 1u) ? 1.f : -1.f;
          const int y = py + tap / 3 - a.pad, x = px + tap % 3 - a.pad;
          const bool ok = y >= 0 && y < a.Hi && x >= 0 && x < a.Wi;
          const int e = ok ? (y * a.Wi + x) * C + c : 0;
          const float xv = ok ? in[e] : 0.f, rv = ok ? rin[e] : 0.f;
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(xv, wv, acc, 0, 0, 0);
          racc = __builtin_amdgcn_mfma_f32_32x32x2f32(rv, wv, racc, 0, 0, 0);
          racc = __builtin_amdgcn_mfma_f32_32x32x2f32(xv, vv, racc, 0, 0, 0);
        }
    }
    // lane holds output n, positions (r/4)*8 + lhalf*4 + r%4.  (All loads before the first store and without conditions: one by one
    // the sixteen took 15000 cycles)
    float bias = 0.f, cz = 0.f, below[16];
    if (EPI == EPI_RELU) {
      bias = a.bias[cur.worker * a.w_wstride + nc];
      const int64_t bi = a.zb_off + nc;
      cz = ((zb[bi >> 5] >> (bi & 31)) & 1u) ? 1.f : -1.f;
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int pr = cur.p0 + wm * 32 + (r >> 2) * 8 + lhalf * 4 + (r & 3);
        below[r] = a.mask[o0 + (int64_t)(pr < npos ? pr : npos - 1) * a.ws.N];
      }
    }
    if (n < a.ws.N) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int pr = cur.p0 + wm * 32 + (r >> 2) * 8 + lhalf * 4 + (r & 3);
        const float c = acc[r] + bias, rc = racc[r] + cz;
        const bool on = EPI == EPI_RELU ? c > 0.f : below[r] > 0.f;
        if (pr < npos) {
          const int64_t o = o0 + (int64_t)pr * a.ws.N;
          a.out[o] = on ? c : 0.f;
          a.rout[o] = on ? rc : 0.f;
        }
      }
    }
    u += stride;
    if (u >= end) return;                                    // (uniform)
    cur = next;
    next = u + stride < end ? place(u + stride) : cur;
    next_w = weights_of(next);
  }
}

// the weights' pieces and signs for the products in both directions: a wave per k-step and 32 outputs
struct FragArgs {
  const float* w; int64_t w_wstride; const uint32_t* zbits; int64_t z_stride, z_off;
  Weights ws[2]; char* frags[2]; int64_t frag_wstride[2];
  uint64_t active_mask;
};
__global__ __launch_bounds__(64) void conv_frags_kernel(FragArgs a) {
  const int dir = blockIdx.z, worker = nth_active_worker(a.active_mask, blockIdx.y);
  const Weights& s = a.ws[dir];
  const int steps = ksteps_of(s.C), lane = threadIdx.x, tile = blockIdx.x / steps, step = blockIdx.x - tile * steps;
  if (tile >= tiles_of(s.N)) return;
  const int tap = step % 9, n = tile * 32 + (lane & 31);
  const uint32_t* zb = a.zbits + worker * a.z_stride;
  float x[8];
  uint32_t v = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int c = step / 9 * KS + (lane >> 5) * 8 + j;
    const bool ok = n < s.N && c < s.C;
    const int64_t o = ok ? (int64_t)n * s.sn + (s.flip ? 8 - tap : tap) * s.st + (int64_t)c * s.sc : 0, b = a.z_off + o;
    x[j] = ok ? a.w[worker * a.w_wstride + o] : 0.f;
    v |= ((zb[b >> 5] >> (b & 31)) & 1u) << j;
  }
  uint32_t o[3][4];
  split_pairs<false, 4>(x, o);
  char* to = a.frags[dir] + worker * a.frag_wstride[dir] + (int64_t)blockIdx.x * kFragBytes + lane * 16;
#pragma unroll
  for (int c = 0; c < 3; ++c) *reinterpret_cast<uint4*>(to + c * 1024) = make_uint4(o[c][0], o[c][1], o[c][2], o[c][3]);
  *reinterpret_cast<uint4*>(to + 3 * 1024) = make_uint4(sign_pair(v, v >> 1), sign_pair(v >> 2, v >> 3), sign_pair(v >> 4, v >> 5), sign_pair(v >> 6, v >> 7));
}

// positions of a block's slab for outputs Ho x Wo in blocks of PB positions
static int64_t slab_entries(int Ho, int Wo, int pb) {
  int64_t rows = (pb - 1 + Wo - 1) / Wo + 1;                 // rows that PB consecutive positions touch at most
  if (rows > Ho) rows = Ho;
  return (rows + 2) * (Wo + 2);
}
static int block_positions(int N) { return N <= 32 ? 256 : 128; }

}  // namespace convf

bool conv_f32_ok(int H, int W, int Cin, int Cout) {
  using namespace convf;
  return slab_entries(H - 2, W - 2, block_positions(Cout)) <= kMostEntries && slab_entries(H, W, block_positions(Cin)) <= kMostEntries;
}
size_t conv_f32_frag_bytes(int N, int C) {
  return (size_t)convf::tiles_of(N) * convf::ksteps_of(C) * convf::kFragBytes;
}

static convf::Weights forward_weights(const ConvF32& c) { return {c.cv.Cout, c.cv.Cin, 9 * c.cv.Cin, c.cv.Cin, 1, 0}; }
static convf::Weights gradient_weights(const ConvF32& c) { return {c.cv.Cin, c.cv.Cout, 1, c.cv.Cin, 9 * c.cv.Cin, 1}; }

hipError_t launch_conv_f32_frags(const ConvF32& c, hipStream_t s) {
  using namespace convf;
  KernelScope ks(KC_GEMM_FWD, s);
  FragArgs a{};
  a.w = c.w; a.w_wstride = c.w_wstride; a.zbits = c.zbits; a.z_stride = c.z_stride; a.z_off = c.z_off;
  a.ws[0] = forward_weights(c); a.ws[1] = gradient_weights(c);
  a.frags[0] = c.fwd_frags; a.frags[1] = c.grad_frags;
  size_t most = 0;
  for (int d = 0; d < 2; ++d) {
    const size_t bytes = conv_f32_frag_bytes(a.ws[d].N, a.ws[d].C);
    a.frag_wstride[d] = (int64_t)bytes;
    most = bytes > most ? bytes : most;
  }
  a.active_mask = c.active_mask;
  hipLaunchKernelGGL(conv_frags_kernel, dim3((unsigned)(most / kFragBytes), (unsigned)active_count(c.active_mask, c.k), 2), dim3(64), 0, s, a);
  return hipGetLastError();
}

// forward: map [B][H][W][Cin] -> [B][H-2][W-2][Cout]; else the gradient map back, masked by the map below
hipError_t launch_conv_f32(const ConvF32& c, bool forward, hipStream_t s) {
  using namespace convf;
  KernelScope ks(forward ? KC_GEMM_FWD : KC_GEMM_DGRAD, s);
  Args a{};
  a.in = c.in; a.rin = c.rin; a.out = c.out; a.rout = c.rout; a.mask = c.mask;
  a.ws = forward ? forward_weights(c) : gradient_weights(c);
  a.frags = forward ? c.fwd_frags : c.grad_frags; a.frag_wstride = (int64_t)conv_f32_frag_bytes(a.ws.N, a.ws.C);
  a.w = c.w; a.w_wstride = c.w_wstride; a.bias = c.bias; a.zbits = c.zbits; a.z_stride = c.z_stride; a.z_off = c.z_off; a.zb_off = c.zb_off;
  a.B = c.B; a.k = c.k; a.active_mask = c.active_mask;
  const int H = c.cv.H, W = c.cv.W;
  a.Hi = forward ? H : H - 2; a.Wi = forward ? W : W - 2; a.Ho = forward ? H - 2 : H; a.Wo = forward ? W - 2 : W; a.pad = forward ? 0 : 2;
  a.in_wstride = (int64_t)c.B * a.Hi * a.Wi * a.ws.C; a.out_wstride = (int64_t)c.B * a.Ho * a.Wo * a.ws.N;
  a.by_wv = (uint32_t)((1ull << 32) / (uint64_t)(a.Wo + 2) + 1);
  const int pb = block_positions(a.ws.N), wn = pb == 256 ? 1 : 2;
  a.blocks = (a.Ho * a.Wo + pb - 1) / pb;
  const int smem = (int)slab_entries(a.Ho, a.Wo, pb) * kPitch;
  const int64_t units = (int64_t)c.B * a.blocks * ((tiles_of(a.ws.N) + wn - 1) / wn) * active_count(c.active_mask, c.k);
  const dim3 grid((unsigned)(units < kBlocks ? (units + 7) / 8 * 8 : kBlocks));
  auto go = [&](auto kern, LdsLimitOnce& lim) -> hipError_t {
    const hipError_t e = lim.raise(reinterpret_cast<const void*>(kern), kMostEntries * kPitch);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, dim3(NT), smem, s, a);
    return hipGetLastError();
  };
  static LdsLimitOnce lim[4];
  if (forward) return wn == 1 ? go(conv3x3_f32<1, EPI_RELU>, lim[0]) : go(conv3x3_f32<2, EPI_RELU>, lim[1]);
  return wn == 1 ? go(conv3x3_f32<1, EPI_MASK>, lim[2]) : go(conv3x3_f32<2, EPI_MASK>, lim[3]);
}

}  // namespace dw
