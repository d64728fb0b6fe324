// Which expert of a token is chosen next, of those that are left: the largest logit, of equal ones the smallest id, and where no
// logit is larger than minus infinity (NaN and minus infinity rank alike, below every number) the smallest id that is left.  So
// whatever a router's logits are, a token gets top_k different ids of [0, E): the grouping that follows takes them as indices.
// Host and device: these are the steps of a lane and the key by which lanes are compared.
#pragma once
#include <hip/hip_runtime.h>

#include <cfloat>
#include <cmath>
#include <cstdint>

namespace rlx {

constexpr float TOPK_GONE = -INFINITY;               // rank of an expert that is taken, or that there is none of
__host__ __device__ __forceinline__ float topk_rank(float logit) { return fmaxf(logit, -FLT_MAX); }

// floats as unsigned integers of the same order, and back
__host__ __device__ __forceinline__ uint32_t float_order_bits(float f) {
  const uint32_t u = __builtin_bit_cast(uint32_t, f);
  return u ^ ((u >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}
__host__ __device__ __forceinline__ float float_from_order_bits(uint32_t o) {
  return __builtin_bit_cast(float, o ^ ((o >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}

// The best of a lane's experts lane, lane + 64, ... as a key: (ordered rank, ~id), the largest of the wave's keys is the choice.
// A lane without an expert left has the rank TOPK_GONE and loses to every lane that has one.
template <int NJ>
__host__ __device__ __forceinline__ uint64_t topk_lane_key(const float (&rank)[NJ], int lane) {
  float br = TOPK_GONE;
  int bi = 0x7FFFFFFF;
#pragma unroll
  for (int j = 0; j < NJ; ++j)
    if (rank[j] > br) { br = rank[j]; bi = lane + 64 * j; }      // ascending id within the lane
  return ((uint64_t)float_order_bits(br) << 32) | (0xFFFFFFFFu - (uint32_t)bi);
}
__host__ __device__ __forceinline__ float topk_key_rank(uint64_t key) { return float_from_order_bits((uint32_t)(key >> 32)); }
__host__ __device__ __forceinline__ int topk_key_id(uint64_t key) { return (int)(0xFFFFFFFFu - (uint32_t)key); }

}  // namespace rlx
