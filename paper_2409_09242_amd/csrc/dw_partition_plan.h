// How the overlap partition lays its scratch out: host arithmetic alone, so that it can be checked for every n without a GPU.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace dw {

// what callers are told: 12 bytes a point, each part rounded up to 256
inline size_t partition_scratch_bytes(int64_t n) {
  const size_t keys = ((size_t)n * 8 + 255) / 256 * 256;
  const size_t rank = ((size_t)n * 4 + 255) / 256 * 256;
  return keys + rank;
}

constexpr int kChunkThreads = 1024, kMaxChunks = 64;         // points of a chunk: one or four a thread; a lane of a wave per chunk
constexpr int64_t kChunksTo = 4 * kMaxChunks * kChunkThreads;            // above this a chunk would need more points or the waves more lanes

struct PartitionPlan {
  int bits, nb;                                              // leading bits of a key that number its bucket; buckets
  int per, chunks;                                           // points of a chunk's thread, chunks (0: five launches)
  size_t bytes;                                              // of scratch that the kernels use
};

inline PartitionPlan partition_plan(int64_t n) {
  PartitionPlan p{};
  if (n <= kChunksTo) {
    p.bits = 5;                                              // 16 to 32 points a bucket (fewer of n < 512)
    while (p.bits < 13 && (n >> (p.bits + 1)) >= 16) p.bits += 1;        // (8192 counters: 32 KB of LDS)
    p.nb = 1 << p.bits;
    p.per = n <= kMaxChunks * kChunkThreads ? 1 : 4;
    p.chunks = (int)((n + kChunkThreads * p.per - 1) / (kChunkThreads * p.per));
    // points [n], then edges [chunks][nb]: with 64 chunks and 16 points a bucket (n = 65536) all of the 12 n bytes
    p.bytes = (size_t)n * 4 + (size_t)p.chunks * p.nb * 2;
  } else {
    p.bits = 13;                                             // 16 to 32 points a bucket
    while ((n >> (p.bits + 1)) >= 16) p.bits += 1;
    p.nb = 1 << p.bits;
    // count [nb], start [nb], slot [n], points [n]: nb <= n / 16
    p.bytes = ((size_t)n * 2 + (size_t)p.nb * 2) * 4;
  }
  return p;
}

}  // namespace dw
