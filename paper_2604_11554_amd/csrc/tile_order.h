// The order in which prefill attention lists its query tiles: by the keys they walk, in buckets of a 1024th of the longest tile's,
// the longest first.  Host and device.
#pragma once
#include <hip/hip_runtime.h>

namespace rlx {

constexpr int TILE_BUCKETS = 1024;
// keys >> tile_shift(longest) < TILE_BUCKETS for keys up to `longest`
__host__ __device__ __forceinline__ int tile_shift(int longest) {
  int bits = 0;
  for (int v = longest; v > 0; v >>= 1) ++bits;
  return bits > 10 ? bits - 10 : 0;
}
// In [0, TILE_BUCKETS) whatever `keys` is: the buckets are counters in LDS, and a place of the list follows from them.
__host__ __device__ __forceinline__ int tile_bucket(int keys, int longest, int shift) {
  const int k = keys < longest ? keys : longest;
  return TILE_BUCKETS - 1 - ((k > 0 ? k : 0) >> shift);
}

}  // namespace rlx
