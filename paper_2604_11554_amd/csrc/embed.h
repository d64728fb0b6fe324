// The embedding that a token row starts from.
#pragma once
#include "common.h"

namespace rlx {

// Embedding of token `tok` -> h[d] in fp32, by the whole workgroup, eight elements per thread (d % 16 == 0); a negative id takes the
// injected row, if any.  An id out of range gives a zero row rather than a stray read.
__device__ __forceinline__ void embed_row(const h16_t* embed, int vocab, int d, int tok, const h16_t* injected, float* h, int dtype) {
  const h16_t* src = nullptr;
  if (tok >= 0 && tok < vocab) src = embed + (size_t)tok * d;
  else if (tok < 0) src = injected;
  for (int i = 8 * (int)threadIdx.x; i < d; i += 8 * (int)blockDim.x) {
    const h16x8 v = src ? load_h16x8(src + i) : zero_h16x8();
    f32x4 lo, hi;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      lo[e] = h16_to_f32((h16_t)(v[e >> 1] >> (16 * (e & 1))), dtype);
      hi[e] = h16_to_f32((h16_t)(v[2 + (e >> 1)] >> (16 * (e & 1))), dtype);
    }
    *reinterpret_cast<f32x4*>(h + i) = lo;
    *reinterpret_cast<f32x4*>(h + i + 4) = hi;
  }
}

}  // namespace rlx
