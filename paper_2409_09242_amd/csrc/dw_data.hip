// Data side of the method on the device (gfx950, wave64).
//
//   partition kernels   Section V-A: one seeded permutation of the n data points, by ranking 64-bit keys; its first
//                       o entries are the shared subset O, the next k blocks of floor((n-o)/k) the private subsets
//                       S_j, and row j of the index array holds D_j = O u S_j (O first, permutation order).
//   gather_kernel       each worker's minibatch: B uniform draws (with replacement) from its own D_j at its local
//                       step, rows and labels copied from the resident data set into the step's input buffers.
//
// The permutation orders the points by (key, index), keys being 64-bit hashes of the index.  The points are put into
// buckets by the keys' leading bits first and ranked within their bucket, so the work is linear in n; exact and independent of
// the order in which threads run.  The gather is a plain row copy bound by HBM bandwidth.
#include <mutex>
#include <type_traits>

#include "dw_internal.h"
#include "dw_partition_plan.h"

// Scratch of dw_overlap_partition_static: what up to DW_STATIC_MAX_POINTS points need (dw_partition_plan.h).  Every device the library
// runs on holds its own copy at its own address until the process ends; host code reaches it only through the address hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) unsigned char scratch[(size_t)DW_STATIC_MAX_POINTS * 12];

namespace dw {

namespace {

constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;

__host__ __device__ inline uint64_t mix64_d(uint64_t x) {      // SplitMix64 output function
  x ^= x >> 30; x *= 0xBF58476D1CE4E5B9ull;
  x ^= x >> 27; x *= 0x94D049BB133111EBull;
  x ^= x >> 31;
  return x;
}

// where the point of rank r in the permutation goes: into every row when it is shared, else into its worker's
// (at most DW_MAX_POINTS points and DW_MAX_K rows: 32-bit places)
__device__ __forceinline__ void partition_place(int32_t* index, int32_t i, int32_t r, int32_t o, int32_t s, int k) {
  const int32_t m = o + s;
  if (r < o) {
    for (int j = 0; j < k; ++j) index[j * m + r] = i;
  } else if (s > 0) {
    const int32_t q = r - o, j = (int32_t)((uint32_t)q / (uint32_t)s);
    if (j < k) index[j * m + o + (q - j * s)] = i;
  }
}
static_assert((int64_t)DW_MAX_POINTS * DW_MAX_K < (1ll << 31), "places fit 32 bits");

// ---- large sets: count, scan, fill, rank by buckets -------------------------------------------------------------------
// Bucket of a point: the leading `bits` bits of its key (bits >= 1).  Keys are computed from the index wherever they are
// needed (two 64-bit multiplies) instead of being stored, so that a point costs 8 bytes of scratch and a bucket 8.

__global__ __launch_bounds__(256) void bucket_clear_kernel(int32_t* count, int nb) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b < nb) count[b] = 0;
}

// slot[i] = how many points had come to i's bucket before it: a place in the bucket, in no particular order
__global__ __launch_bounds__(256) void bucket_count_kernel(int32_t* count, int32_t* slot, int64_t n, int bits, uint64_t k1) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) slot[i] = atomicAdd(&count[mix64_d(k1 + kGamma * (uint64_t)(i + 1)) >> (64 - bits)], 1);
}

// start[b] = points in the buckets before b (one block; nb is a power of two, at least 1024)
__global__ __launch_bounds__(1024) void bucket_scan_kernel(const int32_t* count, int32_t* start, int nb) {
  __shared__ int32_t waves[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = nb / 1024;
  int32_t sum = 0;
  for (int j = 0; j < per; ++j) sum += count[tid * per + j];
  int32_t run = sum;                                           // inclusive over the wave
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t t = __shfl_up(run, off);
    if (lane >= off) run += t;
  }
  if (lane == 63) waves[wave] = run;
  __syncthreads();
  int32_t at = run - sum;
  for (int w = 0; w < wave; ++w) at += waves[w];
  for (int j = 0; j < per; ++j) { start[tid * per + j] = at; at += count[tid * per + j]; }
}

__global__ __launch_bounds__(256) void bucket_fill_kernel(const int32_t* start, const int32_t* slot, int32_t* points,
                                                          int64_t n, int bits, uint64_t k1) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) points[start[mix64_d(k1 + kGamma * (uint64_t)(i + 1)) >> (64 - bits)] + slot[i]] = (int32_t)i;
}

// rank of the point at each place of the bucketed order, and its places in the index array
__global__ __launch_bounds__(256) void bucket_rank_kernel(const int32_t* count, const int32_t* start, const int32_t* points,
                                                          int32_t* index, int64_t n, int bits, uint64_t k1, int64_t o,
                                                          int64_t s, int k) {
  const int64_t at = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (at >= n) return;
  const int32_t i = points[at];
  const uint64_t mine = mix64_d(k1 + kGamma * (uint64_t)((int64_t)i + 1));
  const int64_t b = (int64_t)(mine >> (64 - bits));
  const int32_t first = start[b], len = count[b];
  int32_t r = first;
  for (int32_t j = 0; j < len; ++j) {
    const int32_t other = points[first + j];
    const uint64_t key = mix64_d(k1 + kGamma * (uint64_t)((int64_t)other + 1));
    r += (key < mine || (key == mine && other < i)) ? 1 : 0;
  }
  partition_place(index, i, r, (int32_t)o, (int32_t)s, k);
}

// ---- sets of up to 2^18 points: two launches ---------------------------------------------------------------------------
// The five launches above cost more than their work at such sizes.  A block sorts a chunk of points by bucket in LDS
// and writes them in that order together with where each bucket starts in the chunk; then a wave per bucket adds those starts
// over the chunks (that is the number of points in the buckets before it), collects its points and ranks them.  No counter in
// memory, so nothing is cleared.  Bound by latency: five dependent trips to memory.  n = 60000: the kernels 10 us, the whole call 26 (five launches: 28 and 43; buckets of
// 64 to 128 points with four waves each 39, 20 of them comparing keys).

// chunk c: the CH points from c * CH on, at points[c * CH ...] by bucket; edge[c * nb + b]: the first of bucket b
template <int PER>
__global__ __launch_bounds__(kChunkThreads) void chunk_sort_kernel(uint16_t* edge, int32_t* points, int64_t n, int bits, uint64_t k1) {
  constexpr int CH = kChunkThreads * PER;
  extern __shared__ int32_t first[];                           // [nb]: counts, then places
  __shared__ int32_t waves[kChunkThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nb = 1 << bits;
  uint16_t* edges = edge + (int64_t)blockIdx.x * nb;
  const int64_t i0 = (int64_t)blockIdx.x * CH;
  for (int b = tid; b < nb; b += kChunkThreads) first[b] = 0;
  __syncthreads();
  int bucket[PER], slot[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int64_t i = i0 + j * kChunkThreads + tid;
    bucket[j] = i < n ? (int)(mix64_d(k1 + kGamma * (uint64_t)(i + 1)) >> (64 - bits)) : -1;
    slot[j] = bucket[j] >= 0 ? atomicAdd(&first[bucket[j]], 1) : 0;      // a place in the bucket, in no particular order
  }
  __syncthreads();
  const int per = (nb + kChunkThreads - 1) / kChunkThreads;    // buckets of a thread
  int32_t sum = 0;
  for (int j = 0; j < per; ++j) sum += tid * per + j < nb ? first[tid * per + j] : 0;
  int32_t run = sum;                                           // inclusive over the wave
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t t = __shfl_up(run, off);
    if (lane >= off) run += t;
  }
  if (lane == 63) waves[wave] = run;
  __syncthreads();
  int32_t at = run - sum;
  for (int w = 0; w < wave; ++w) at += waves[w];
  for (int j = 0; j < per && tid * per + j < nb; ++j) {
    const int b = tid * per + j;
    const int32_t c = first[b];
    first[b] = at;
    edges[b] = (uint16_t)at;
    at += c;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < PER; ++j)
    if (bucket[j] >= 0) points[i0 + first[bucket[j]] + slot[j]] = (int32_t)(i0 + j * kChunkThreads + tid);
}

// a wave per bucket: collect its points (a lane per chunk), rank them, place them
template <int PER>
__global__ __launch_bounds__(64) void chunk_rank_kernel(const uint16_t* edge, const int32_t* points, int64_t n, int nb, int chunks,
                                                        int32_t* index, uint64_t k1, int32_t o, int32_t s, int k) {
  constexpr int CH = kChunkThreads * PER, T = 64;
  static_assert(kMaxChunks <= T, "a lane per chunk");
  __shared__ uint64_t key[T];
  __shared__ int32_t point[T];
  const int lane = threadIdx.x, b = blockIdx.x;
  // this lane's chunk: where the bucket starts in it, and how many points it has (the last bucket ends where the chunk does)
  const uint16_t* e = edge + (int64_t)lane * nb + b;
  const int left = (int)(n - (int64_t)lane * CH), end = left < CH ? left : CH;
  const int lo = lane < chunks ? e[0] : 0, len = lane < chunks ? (b + 1 < nb ? e[1] : end) - lo : 0;
  int32_t run = len, rank0 = lo;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t t = __shfl_up(run, off);
    if (lane >= off) run += t;
    rank0 += __shfl_xor(rank0, off);
  }
  const int32_t total = __shfl(run, 63), at = run - len;       // at: the chunk's first point in the bucket's list
  const int32_t* mine = points + (int64_t)lane * CH + lo;
  auto stage = [&](int from) {                                 // list entries from .. from + T - 1 into LDS
    for (int j = from > at ? from - at : 0; j < len && at + j < from + T; ++j) {
      const int32_t i = mine[j];
      point[at + j - from] = i;
      key[at + j - from] = mix64_d(k1 + kGamma * (uint64_t)((int64_t)i + 1));
    }
  };
  // (a list longer than the wave, more than five standard deviations above the mean, takes turns; two points never have the same key:
  // the mixing function and the multiplication by an odd number are one to one)
  for (int own = 0; own < total; own += T) {
    __syncthreads();
    stage(own);
    __syncthreads();
    const bool ok = own + lane < total;
    const uint64_t me = ok ? key[lane] : 0;
    const int32_t i = ok ? point[lane] : 0;
    int32_t r = rank0;
    for (int other = 0; other < total; other += T) {
      if (total > T) {
        __syncthreads();
        stage(other);
        __syncthreads();
      }
      const int m = total - other < T ? total - other : T;
#pragma unroll 8
      for (int j = 0; j < m; ++j) r += key[j] < me ? 1 : 0;
    }
    if (ok) partition_place(index, i, r, o, s, k);
  }
}

struct GatherKeys { uint64_t key[DW_MAX_K]; };

// block (b, j): draw b of worker j, one row of row_vecs 16-byte pieces
__global__ __launch_bounds__(256) void gather_kernel(const uint4* data, const int32_t* labels, const int32_t* index,
                                                     int64_t n, int64_t m, int row_vecs, int B, GatherKeys keys,
                                                     uint64_t active_mask, uint4* x, int32_t* y) {
  const int j = blockIdx.y, b = blockIdx.x;
  if (!((active_mask >> j) & 1ull)) return;
  const uint64_t u = mix64_d(keys.key[j] + kGamma * (uint64_t)(b + 1));
  const int64_t pos = (int64_t)__umul64hi(u, (uint64_t)m);     // floor(u * m / 2^64)
  const int64_t idx = index[(int64_t)j * m + pos];
  const bool ok = idx >= 0 && idx < n;                         // an index outside the data set yields a zero row
  uint4* dst = x + ((int64_t)j * B + b) * row_vecs;
  if (ok) {
    const uint4* src = data + idx * row_vecs;
    for (int v = threadIdx.x; v < row_vecs; v += 256) dst[v] = src[v];
    if (threadIdx.x == 0) y[(int64_t)j * B + b] = labels[idx];
  } else {
    for (int v = threadIdx.x; v < row_vecs; v += 256) dst[v] = make_uint4(0u, 0u, 0u, 0u);
    if (threadIdx.x == 0) y[(int64_t)j * B + b] = -1;
  }
}

}  // namespace

hipError_t launch_partition(int64_t n, int64_t o, int k, uint64_t seed, int32_t* index, void* scratch, hipStream_t s) {
  const int64_t sz = (n - o) / k;
  const uint64_t k1 = mix64_d(seed);
  const PartitionPlan plan = partition_plan(n);
  const int bits = plan.bits, nb = plan.nb;
  if (plan.chunks > 0) {
    auto launch = [&](auto per) {
      constexpr int PER = decltype(per)::value;
      int32_t* points = reinterpret_cast<int32_t*>(scratch);
      uint16_t* edge = reinterpret_cast<uint16_t*>(points + n);
      hipLaunchKernelGGL(chunk_sort_kernel<PER>, dim3((unsigned)plan.chunks), dim3(kChunkThreads), nb * (int)sizeof(int32_t), s, edge, points, n,
                         bits, k1);
      hipLaunchKernelGGL(chunk_rank_kernel<PER>, dim3((unsigned)nb), dim3(64), 0, s, edge, points, n, nb, plan.chunks, index, k1, (int32_t)o,
                         (int32_t)sz, k);
    };
    if (plan.per == 1) launch(std::integral_constant<int, 1>{}); else launch(std::integral_constant<int, 4>{});
    return hipGetLastError();
  }
  int32_t* count = reinterpret_cast<int32_t*>(scratch);
  int32_t* start = count + nb;
  int32_t* slot = start + nb;
  int32_t* points = slot + n;
  const unsigned blocks = (unsigned)((n + 255) / 256);
  hipLaunchKernelGGL(bucket_clear_kernel, dim3((unsigned)(nb / 256)), dim3(256), 0, s, count, nb);
  hipLaunchKernelGGL(bucket_count_kernel, dim3(blocks), dim3(256), 0, s, count, slot, n, bits, k1);
  hipLaunchKernelGGL(bucket_scan_kernel, dim3(1), dim3(1024), 0, s, count, start, nb);
  hipLaunchKernelGGL(bucket_fill_kernel, dim3(blocks), dim3(256), 0, s, start, slot, points, n, bits, k1);
  hipLaunchKernelGGL(bucket_rank_kernel, dim3(blocks), dim3(256), 0, s, count, start, points, index, n, bits, k1, o, sz, k);
  return hipGetLastError();
}

hipError_t launch_gather(const void* data, const int32_t* labels, const int32_t* index, int64_t n, int64_t m,
                         int row_bytes, int B, int k, const uint64_t* keys_host, uint64_t active_mask, void* x,
                         int32_t* y, hipStream_t s) {
  KernelScope ks(KC_GATHER, s);
  GatherKeys keys;
  for (int i = 0; i < DW_MAX_K; ++i) keys.key[i] = i < k ? keys_host[i] : 0;
  hipLaunchKernelGGL(gather_kernel, dim3((unsigned)B, (unsigned)k), dim3(256), 0, s,
                     reinterpret_cast<const uint4*>(data), labels, index, n, m, row_bytes / 16, B, keys, active_mask,
                     reinterpret_cast<uint4*>(x), y);
  return hipGetLastError();
}

// device address of `scratch` on the current device, looked up once per device
hipError_t static_scratch(void** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptr[kMaxDevices] = {nullptr};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    ptr[dev] = p;
  }
  *out = ptr[dev];
  return hipSuccess;
}

}  // namespace dw

extern "C" int64_t dw_overlap_partition_static(int64_t n, int64_t o, int k, uint64_t seed, int32_t* d_index,
                                               void* stream) {
  if (n < 1 || o < 0 || o > n || k < 1 || k > DW_MAX_K) return DW_ERR_ARG;
  if (n > DW_STATIC_MAX_POINTS) return DW_ERR_TOO_LARGE;
  static_assert(sizeof(scratch) % 256 == 0, "the rank array starts at a multiple of 256 bytes");
  if (dw::partition_scratch_bytes(n) > sizeof(scratch)) return DW_ERR_TOO_LARGE;
  const int64_t sz = (n - o) / k;
  if (!d_index && o + sz > 0) return DW_ERR_NULL;
  void* d_scratch = nullptr;
  hipError_t e = dw::static_scratch(&d_scratch);
  if (e == hipSuccess) e = dw::launch_partition(n, o, k, seed, d_index, d_scratch, (hipStream_t)stream);
  if (e != hipSuccess) return dw::note_hip_error(e);
  return sz;
}
