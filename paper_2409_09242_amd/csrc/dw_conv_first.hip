// The first 3x3 convolution of the front end where the image has one channel: forward with its R-companion, and weight gradient
// (Section VI's model, Section IV-B).  The image's own companion is zero, so
//   S = bias + sum over nine taps of W x,  RS = c + sum of V x,  gW = sum over positions of d x,  HzW = sum of Rd x.
//
// Nine products an output are no work for the matrix cores: what bounds both is writing or reading two maps of N channels.  A thread owns
// four channels and a column of the map and goes down its rows, so that a wave moves 1 KB pieces of the two maps, three
// new pixels a row replace three old ones, and the taps (forward) or the 80 sums (gradient) stay in registers.  Products and sums are in
// 64 bits, which cost what 32 cost here: one rounding an output, whatever the number of positions.
// A minibatch's gradient is added up over a block in LDS and over blocks in their order (conv_first_sum_kernel).
// Eight workers, 64 images of 28 x 28, 32 channels: patches 22 and forward 31 (as a product of tiles) -> 28 us, 89 MB written; weight
// gradient 66 and sum of its slices 9 -> 21 and 5.  Waits for all that is on its way instead of one row's pixels: forward 35; one row on its way
// instead of two: gradient 28.  Columns in two, three or four strips: each 1 to 2 us slower.  More input channels have more taps than registers
// hold: they go through patches.
#include "dw_internal.h"
#include "dw_head_math.h"

namespace dw {

namespace conv1 {

constexpr int NT = 256, COLS = NT / 8, CH = 32;              // columns and channels of a block
constexpr int kSums = 20;                                    // of a channel: nine of gW, nine of HzW, the two bias gradients

struct Args {
  const float* x; int64_t x_wstride;                         // images [B][H][W]
  float* a; float* ra; int64_t a_wstride;                    // forward: outputs [B][Ho][Wo][N]; gradient: d, Rd (read)
  const float* w; int64_t w_wstride; const float* bias;
  const uint32_t* zbits; int64_t z_stride, z_off, zb_off;
  int B, W, Ho, Wo, N, K, rows, tasks, blocks;               // rows a thread walks; tasks: strips x images x columns; blocks of them
  uint64_t active_mask;
  double* part;                                              // [worker][block][N][kSums]
  float* g; float* hz; float* gb; float* hzb;                // of worker 0, stride w_wstride
};

struct Place { const float* px; int64_t o; int rows; };      // first pixel, first output, rows to walk
__device__ __forceinline__ Place place_of(const Args& a, int task, int worker, int c) {
  const int per = a.B * a.Wo, strip = task / per, r = task - strip * per, b = r / a.Wo, x = r - b * a.Wo, y0 = strip * a.rows;
  const int H = a.Ho + 2;
  return {a.x + worker * a.x_wstride + ((int64_t)b * H + y0) * a.W + x, worker * a.a_wstride + (((int64_t)b * a.Ho + y0) * a.Wo + x) * a.N + c,
          a.rows < a.Ho - y0 ? a.rows : a.Ho - y0};
}

__global__ __launch_bounds__(NT, 2) void conv_first_kernel(Args a) {
  const int worker = nth_active_worker(a.active_mask, blockIdx.z), c = blockIdx.y * CH + (threadIdx.x & 7) * 4;
  const int task = blockIdx.x * COLS + (threadIdx.x >> 3);
  if (task >= a.tasks || c >= a.N) return;
  const Place at = place_of(a, task, worker, c);
  const uint32_t* zb = a.zbits + worker * a.z_stride;
  auto sign = [&](int64_t bit) { return ((zb[bit >> 5] >> (bit & 31)) & 1u) ? 1.0 : -1.0; };
  double w[4][9], v[4][9], bias[4], cz[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    bias[q] = a.bias[worker * a.w_wstride + c + q];
    cz[q] = sign(a.zb_off + c + q);
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int64_t o = (int64_t)(c + q) * a.K + t;
      w[q][t] = a.w[worker * a.w_wstride + o];
      v[q][t] = sign(a.z_off + o);
    }
  }
  double p[9];
#pragma unroll
  for (int t = 0; t < 6; ++t) p[3 + t] = at.px[(t / 3) * a.W + t % 3];
  struct Row { float n[3]; } even, odd;                      // two rows on their way
  auto fetch = [&](Row& to, int y) {
    const float* px = at.px + (int64_t)(2 + (y < at.rows ? y : at.rows - 1)) * a.W;
    to.n[0] = px[0]; to.n[1] = px[1]; to.n[2] = px[2];
  };
  auto step = [&](Row& now, int y) {
#pragma unroll
    for (int t = 0; t < 6; ++t) p[t] = p[3 + t];
    p[6] = now.n[0]; p[7] = now.n[1]; p[8] = now.n[2];
    fetch(now, y + 2);
    float s[4], rs[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      double t0 = bias[q], t1 = cz[q];
#pragma unroll
      for (int t = 0; t < 9; ++t) { t0 = fma(w[q][t], p[t], t0); t1 = fma(v[q][t], p[t], t1); }
      s[q] = (float)t0;
      const bool on = s[q] > 0.f;
      s[q] = on ? s[q] : 0.f;
      rs[q] = on ? (float)t1 : 0.f;
    }
    const int64_t o = at.o + (int64_t)y * a.Wo * a.N;
    *reinterpret_cast<float4*>(a.a + o) = make_float4(s[0], s[1], s[2], s[3]);
    *reinterpret_cast<float4*>(a.ra + o) = make_float4(rs[0], rs[1], rs[2], rs[3]);
  };
  // (The first two rows stand before the loop so that a wait in it is for the row's pixels alone, not for the stores behind them.)
  fetch(even, 0); fetch(odd, 1);
  int y = 0;
  if (at.rows > 1) {
    step(even, 0); step(odd, 1);
    for (y = 2; y + 1 < at.rows; y += 2) { step(even, y); step(odd, y + 1); }
  }
  if (y < at.rows) step(even, y);
}

// sums of two values over the halves of a wave (rows of it: ROWS), a's in the lower lanes (even rows), b's in the others
template <bool ROWS>
__device__ __forceinline__ double add_swapped(double x, double y) {
  const uint2 a = __builtin_bit_cast(uint2, x), b = __builtin_bit_cast(uint2, y);
  uint2 p, q;
  if constexpr (ROWS) {
    const auto l = __builtin_amdgcn_permlane16_swap(a.x, b.x, false, false), h = __builtin_amdgcn_permlane16_swap(a.y, b.y, false, false);
    p = make_uint2(l[0], h[0]); q = make_uint2(l[1], h[1]);
  } else {
    const auto l = __builtin_amdgcn_permlane32_swap(a.x, b.x, false, false), h = __builtin_amdgcn_permlane32_swap(a.y, b.y, false, false);
    p = make_uint2(l[0], h[0]); q = make_uint2(l[1], h[1]);
  }
  return __builtin_bit_cast(double, p) + __builtin_bit_cast(double, q);
}

__global__ __launch_bounds__(NT, 2) void conv_first_grad_kernel(Args a) {
  __shared__ double red[NT / 64][4][kSums][8];
  const int worker = nth_active_worker(a.active_mask, blockIdx.z), lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = blockIdx.y * CH + (lane & 7) * 4, task = blockIdx.x * COLS + (threadIdx.x >> 3);
  const bool mine = task < a.tasks && c < a.N;
  Place at = place_of(a, mine ? task : 0, worker, mine ? c : 0);
  if (!mine) at.rows = 0;
  double sum[4 * kSums];                                     // [channel][sum]
#pragma unroll
  for (int i = 0; i < 4 * kSums; ++i) sum[i] = 0.0;
  double p[9];
#pragma unroll
  for (int t = 0; t < 6; ++t) p[3 + t] = at.px[(t / 3) * a.W + t % 3];
  struct Row { float n[3]; float4 d, r; } even, odd;         // two rows on their way (further ones than the last: the last again)
  const int64_t row = (int64_t)a.Wo * a.N;
  auto fetch = [&](Row& to, int y) {
    const int at_y = y < at.rows ? y : at.rows > 0 ? at.rows - 1 : 0;
    const float* px = at.px + (int64_t)(2 + at_y) * a.W;
    to.n[0] = px[0]; to.n[1] = px[1]; to.n[2] = px[2];
    to.d = *reinterpret_cast<const float4*>(a.a + at.o + at_y * row);
    to.r = *reinterpret_cast<const float4*>(a.ra + at.o + at_y * row);
  };
  auto step = [&](Row& now, int y) {
#pragma unroll
    for (int t = 0; t < 6; ++t) p[t] = p[3 + t];
    p[6] = now.n[0]; p[7] = now.n[1]; p[8] = now.n[2];
    const double d[4] = {now.d.x, now.d.y, now.d.z, now.d.w}, rd[4] = {now.r.x, now.r.y, now.r.z, now.r.w};
    fetch(now, y + 2);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      double* s = sum + q * kSums;
#pragma unroll
      for (int t = 0; t < 9; ++t) { s[t] = fma(d[q], p[t], s[t]); s[9 + t] = fma(rd[q], p[t], s[9 + t]); }
      s[18] += d[q]; s[19] += rd[q];
    }
  };
  fetch(even, 0); fetch(odd, 1);
  int y = 0;
  for (; y + 1 < at.rows; y += 2) { step(even, y); step(odd, y + 1); }
  if (y < at.rows) step(even, y);
  // a wave's eight columns: row r of its lanes ends up with channel r's sums
#pragma unroll
  for (int i = 0; i < 2 * kSums; ++i) sum[i] = add_swapped<false>(sum[i], sum[i + 2 * kSums]);
#pragma unroll
  for (int i = 0; i < kSums; ++i) {
    double t = add_swapped<true>(sum[i], sum[i + kSums]);
    t += row_move<kRowTurn + 8>(t);
    if ((lane & 8) == 0) red[wave][lane >> 4][i][lane & 7] = t;
  }
  __syncthreads();
  double* to = a.part + ((int64_t)worker * a.blocks + blockIdx.x) * a.N * kSums;
  for (int i = threadIdx.x; i < CH * kSums; i += NT) {
    const int ch = i / kSums, e = i - ch * kSums, n = blockIdx.y * CH + ch;
    if (n < a.N) to[(int64_t)n * kSums + e] = (red[0][ch & 3][e][ch >> 2] + red[1][ch & 3][e][ch >> 2]) + (red[2][ch & 3][e][ch >> 2] + red[3][ch & 3][e][ch >> 2]);
  }
}

// a wave per channel: three groups of lanes add up every third block's sums
__global__ __launch_bounds__(64) void conv_first_sum_kernel(Args a) {
  const int worker = nth_active_worker(a.active_mask, blockIdx.y), n = blockIdx.x, lane = threadIdx.x;
  const int third = lane / kSums, e = lane - third * kSums;
  const double* from = a.part + ((int64_t)worker * a.blocks * a.N + n) * kSums + e;
  double t = 0.0;
  if (third < 3) {
    constexpr int U = 6;
    for (int b = third; b < a.blocks; b += 3 * U) {
      double x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) { const int at = b + 3 * u; x[u] = at < a.blocks ? from[(int64_t)at * a.N * kSums] : 0.0; }
#pragma unroll
      for (int u = 0; u < U; ++u) t += x[u];
    }
  }
  const double t1 = __shfl(t, e + kSums), t2 = __shfl(t, e + 2 * kSums);
  t = t + t1 + t2;
  const int64_t w = worker * a.w_wstride;
  if (lane < 9) a.g[w + (int64_t)n * a.K + lane] = (float)t;
  else if (lane < 18) a.hz[w + (int64_t)n * a.K + lane - 9] = (float)t;
  else if (lane == 18) a.gb[w + n] = (float)t;
  else if (lane == 19) a.hzb[w + n] = (float)t;
  else if (lane < 20 + a.K - 9) a.g[w + (int64_t)n * a.K + lane - 11] = 0.f;      // the columns that fill a row of W up
  else if (lane < 20 + 2 * (a.K - 9)) a.hz[w + (int64_t)n * a.K + lane - 11 - (a.K - 9)] = 0.f;
}

// Rows a thread walks: all of a column, or fewer where that leaves compute units without a block
static void split(Args& a, int k) {
  const int64_t cols = (int64_t)a.B * a.Wo, blocks = (cols + COLS - 1) / COLS * ((a.N + CH - 1) / CH) * k;
  int64_t strips = (256 + blocks - 1) / blocks;
  if (strips > (a.Ho + 3) / 4) strips = (a.Ho + 3) / 4;
  a.rows = (int)((a.Ho + strips - 1) / strips);
  strips = (a.Ho + a.rows - 1) / a.rows;
  a.tasks = (int)(strips * cols);
  a.blocks = (a.tasks + COLS - 1) / COLS;
}

static Args args_of(const ConvF32& c) {
  Args a{};
  a.B = c.B; a.W = c.cv.W; a.Ho = c.cv.H - 2; a.Wo = c.cv.W - 2; a.N = c.cv.Cout; a.K = 12;
  split(a, c.k);
  return a;
}

}  // namespace conv1

bool conv_first_ok(const ConvF32& c) {
  return c.cv.Cin == 1 && c.cv.Cout % 4 == 0 && (int64_t)c.B * c.cv.H * c.cv.W < (1ll << 30) && (c.cv.Cout + conv1::CH - 1) / conv1::CH <= 65535;
}
size_t conv_first_part_bytes(const ConvF32& c) {
  return (size_t)c.k * conv1::args_of(c).blocks * c.cv.Cout * conv1::kSums * sizeof(double);
}

static conv1::Args first_args(const ConvF32& c) {
  conv1::Args a = conv1::args_of(c);
  a.x = c.in; a.x_wstride = (int64_t)c.B * c.cv.H * c.cv.W; a.a_wstride = (int64_t)c.B * a.Ho * a.Wo * a.N;
  a.w = c.w; a.w_wstride = c.w_wstride; a.bias = c.bias;
  a.zbits = c.zbits; a.z_stride = c.z_stride; a.z_off = c.z_off; a.zb_off = c.zb_off; a.active_mask = c.active_mask;
  return a;
}

hipError_t launch_conv_first(const ConvF32& c, hipStream_t s) {
  KernelScope ks(KC_GEMM_FWD, s);
  conv1::Args a = first_args(c);
  a.a = c.out; a.ra = c.rout;
  const dim3 grid((unsigned)a.blocks, (unsigned)((a.N + conv1::CH - 1) / conv1::CH), (unsigned)active_count(c.active_mask, c.k));
  hipLaunchKernelGGL(conv1::conv_first_kernel, grid, dim3(conv1::NT), 0, s, a);
  return hipGetLastError();
}

// d, Rd in c.out, c.rout; the gradients of W and of the bias go to g, hz and gb, hzb (worker 0, stride w_wstride)
hipError_t launch_conv_first_grad(const ConvF32& c, double* part, float* g, float* hz, float* gb, float* hzb, hipStream_t s) {
  KernelScope ks(KC_GEMM_WGRAD, s);
  conv1::Args a = first_args(c);
  a.a = c.out; a.ra = c.rout; a.part = part; a.g = g; a.hz = hz; a.gb = gb; a.hzb = hzb;
  const unsigned active = (unsigned)active_count(c.active_mask, c.k);
  hipLaunchKernelGGL(conv1::conv_first_grad_kernel, dim3((unsigned)a.blocks, (unsigned)((a.N + conv1::CH - 1) / conv1::CH), active),
                     dim3(conv1::NT), 0, s, a);
  hipLaunchKernelGGL(conv1::conv_first_sum_kernel, dim3((unsigned)a.N, active), dim3(64), 0, s, a);
  return hipGetLastError();
}

}  // namespace dw
