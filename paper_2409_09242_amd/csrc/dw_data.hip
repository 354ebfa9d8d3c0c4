// Data side of the method on the device (gfx950, wave64).
//
//   partition kernels   Section V-A: one seeded permutation of the n data points, by ranking 64-bit keys; its first
//                       o entries are the shared subset O, the next k blocks of floor((n-o)/k) the private subsets
//                       S_j, and row j of the index array holds D_j = O u S_j (O first, permutation order).
//   gather_kernel       each worker's minibatch: B uniform draws (with replacement) from its own D_j at its local
//                       step, rows and labels copied from the resident data set into the step's input buffers.
//
// The permutation orders the points by (key, index), keys being 64-bit hashes of the index.  A large set is put into
// buckets by the keys' leading bits first (about 16 to 32 points each) and a point is ranked within its bucket, so the
// work is linear in n; a small one is ranked by comparing every pair.  Both are exact and independent of the order in
// which threads run.  The gather is a plain row copy bound by HBM bandwidth.
#include <mutex>

#include "dw_internal.h"

// Scratch of dw_overlap_partition_static: keys and ranks of up to DW_STATIC_MAX_POINTS points, in the layout
// partition_scratch_bytes describes.  Every device the library runs on holds its own copy at its own address until the
// process ends; host code reaches it only through the address hipGetSymbolAddress returns for the current device.
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

__global__ __launch_bounds__(256) void partition_keys_kernel(uint64_t* keys, int32_t* rank, int64_t n, uint64_t k1) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  keys[i] = mix64_d(k1 + kGamma * (uint64_t)(i + 1));
  rank[i] = 0;
}

// rank[i] += number of points j of this block row's slice with (key_j, j) < (key_i, i)
__global__ __launch_bounds__(256) void partition_rank_kernel(const uint64_t* keys, int32_t* rank, int64_t n,
                                                             int64_t slice) {
  __shared__ uint64_t tile[256];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const uint64_t mine = i < n ? keys[i] : 0;
  const int64_t j0 = (int64_t)blockIdx.y * slice;
  const int64_t j1 = j0 + slice < n ? j0 + slice : n;
  int32_t cnt = 0;
  for (int64_t base = j0; base < j1; base += 256) {            // uniform trip count: every thread reaches the barriers
    const int64_t j = base + threadIdx.x;
    __syncthreads();
    tile[threadIdx.x] = j < j1 ? keys[j] : ~0ull;
    __syncthreads();
    const int lim = (int)(j1 - base < 256 ? j1 - base : 256);
    for (int t = 0; t < lim; ++t) {
      const uint64_t other = tile[t];
      cnt += (other < mine || (other == mine && base + t < i)) ? 1 : 0;
    }
  }
  if (i < n && cnt != 0) atomicAdd(&rank[i], cnt);
}

// where the point of rank r in the permutation goes: into every row when it is shared, else into its worker's
__device__ __forceinline__ void partition_place(int32_t* index, int64_t i, int64_t r, int64_t o, int64_t s, int k) {
  const int64_t m = o + s;
  if (r < o) {
    for (int j = 0; j < k; ++j) index[(int64_t)j * m + r] = (int32_t)i;
  } else if (s > 0) {
    const int64_t q = r - o;
    const int64_t j = q / s;
    if (j < k) index[j * m + o + (q - j * s)] = (int32_t)i;
  }
}

__global__ __launch_bounds__(256) void partition_scatter_kernel(const int32_t* rank, int32_t* index, int64_t n,
                                                                int64_t o, int64_t s, int k) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) partition_place(index, i, rank[i], o, s, k);
}

// ---- the same through buckets: count, scan, fill, rank ---------------------------------------------------------------
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
  partition_place(index, i, r, o, s, k);
}

// Buckets are used from the size on that has scratch for the least number of them, 8 n + 8 * 1024 <= 12 n bytes: there
// five short launches take as long as comparing every pair (whole call 33 us against 43 at n = 4000, 43 at n = 2000 for
// the pairs), and then the pairs grow with n^2 (n = 60000: 0.945 ms -> 43 us, of which the kernels 28: counting and ranking
// 10 each, bound by the atomics' and the bucket walk's latency; n = 2^21: 914 -> 0.41 ms).
constexpr int64_t kBucketFrom = 2048;

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

size_t partition_scratch_bytes(int64_t n) {
  const size_t keys = ((size_t)n * 8 + 255) / 256 * 256;
  const size_t rank = ((size_t)n * 4 + 255) / 256 * 256;
  return keys + rank;
}

hipError_t launch_partition(int64_t n, int64_t o, int k, uint64_t seed, int32_t* index, void* scratch, hipStream_t s) {
  const int64_t sz = (n - o) / k;
  if (n >= kBucketFrom) {
    int bits = 10;                                             // at least 1024 buckets, then 16 to 32 points a bucket
    while ((n >> (bits + 1)) >= 16) bits += 1;
    const int nb = 1 << bits;
    // 8 n + 8 nb bytes, nb <= n / 16: within the 12 n of partition_scratch_bytes
    int32_t* count = reinterpret_cast<int32_t*>(scratch);
    int32_t* start = count + nb;
    int32_t* slot = start + nb;
    int32_t* points = slot + n;
    const unsigned blocks = (unsigned)((n + 255) / 256);
    const uint64_t k1 = mix64_d(seed);
    hipLaunchKernelGGL(bucket_clear_kernel, dim3((unsigned)(nb / 256)), dim3(256), 0, s, count, nb);
    hipLaunchKernelGGL(bucket_count_kernel, dim3(blocks), dim3(256), 0, s, count, slot, n, bits, k1);
    hipLaunchKernelGGL(bucket_scan_kernel, dim3(1), dim3(1024), 0, s, count, start, nb);
    hipLaunchKernelGGL(bucket_fill_kernel, dim3(blocks), dim3(256), 0, s, start, slot, points, n, bits, k1);
    hipLaunchKernelGGL(bucket_rank_kernel, dim3(blocks), dim3(256), 0, s, count, start, points, index, n, bits, k1, o, sz, k);
    return hipGetLastError();
  }
  uint64_t* keys = reinterpret_cast<uint64_t*>(scratch);
  int32_t* rank = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(scratch) + ((size_t)n * 8 + 255) / 256 * 256);
  const unsigned nb = (unsigned)((n + 255) / 256);
  hipLaunchKernelGGL(partition_keys_kernel, dim3(nb), dim3(256), 0, s, keys, rank, n, mix64_d(seed));
  // enough block rows to fill the chip when n is small; each covers a slice of the points compared against
  int64_t rows = 2048 / nb;
  if (rows < 1) rows = 1;
  if (rows > nb) rows = nb;
  int64_t slice = ((n + rows - 1) / rows + 255) / 256 * 256;
  rows = (n + slice - 1) / slice;
  hipLaunchKernelGGL(partition_rank_kernel, dim3(nb, (unsigned)rows), dim3(256), 0, s, keys, rank, n, slice);
  hipLaunchKernelGGL(partition_scatter_kernel, dim3(nb), dim3(256), 0, s, rank, index, n, o, sz, k);
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
