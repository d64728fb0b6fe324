// Last stage of a step: merge the LM-head tiles' (max, sumexp, best perturbed score,
// argbest) partials in tile order, apply teacher forcing and the length cap, score the
// emitted token (log-softmax of the temperature-scaled logits) and update the
// per-sequence state (token, cached length, finished flag).
#include "kernels.h"

namespace rlx {
namespace {

struct Part { float m, s, best; int besti; };

// Equal perturbed scores go to the smaller token id whatever the order of the merges.
__device__ __forceinline__ Part part_merge(Part a, Part b) {
  Part r;
  float mn = fmaxf(a.m, b.m);
  float ea = (a.m == -INFINITY) ? 0.f : __expf(a.m - mn);
  float eb = (b.m == -INFINITY) ? 0.f : __expf(b.m - mn);
  r.m = mn; r.s = a.s * ea + b.s * eb;
  const bool take_b = b.best > a.best || (b.best == a.best && b.besti < a.besti);
  r.best = take_b ? b.best : a.best;
  r.besti = take_b ? b.besti : a.besti;
  return r;
}

// What bounds it: round trips, of which only the emitted token's weights wait for another one's answer, and they only where the token is
// drawn and not given.  Everything else is requested at once, and the tree over the threads stays in their waves.  us per launch, each
// load where it was first used -> now: two-layer policy, tokens given 5.4 -> 4.2, drawn 5.3 -> 4.3; 151 936 ids, 1 row 8.5 -> 7.2 and
// 8.5 -> 7.7, 64 rows 10.7 -> 9.0 and 9.9 -> 9.1, 256 rows 11.9 -> 9.4 and 11.6 -> 9.4.
// SCORE: many rows, some with nothing to score, which leave before they ask for anything; row and weights come behind the parts.  us for
// 896 scored rows, 608, and the same with a third of them scored: each load where it was first used 15.0, 12.8, 9.7, 9.2; everything at
// once 15.8, 13.8, 12.6, 10.8; now 15.7, 12.7, 10.0, 9.5.
template <bool SCORE>
__global__ __launch_bounds__(256) void sample_finalize_kernel(FinalizeArgs a) {
  __shared__ Part sh[4];
  __shared__ float dsh[4];
  const int r = blockIdx.x, tid = (int)threadIdx.x;
  const int forced = a.forced ? a.forced[r] : -1;
  const bool given = forced >= 0 && forced < a.vocab;
  if (SCORE && !given) {                    // nothing to score at this position
    if (tid == 0) a.out_logprobs[r] = 0.f;
    return;
  }
  const float temp = a.temperature[a.row_seq ? a.row_seq[r] : r];
  const uint8_t sample_on = SCORE ? 1 : a.sample_on[r];
  const int pos = SCORE ? 0 : a.sample_pos[r], max_ctx_len = SCORE ? 0x7FFFFFFF : a.max_ctx_len[r];
  const f32x4* base = reinterpret_cast<const f32x4*>(a.part + (size_t)r * a.n_parts * 4);
  f32x4 q[8];
  auto load_parts = [&](int t0) {
#pragma unroll
    for (int u = 0; u < 8; ++u) q[u] = base[min(t0 + u * 256 + tid, a.n_parts - 1)];
  };
  load_parts(0);
  // the row's and the emitted token's features: eight consecutive k are one 16-byte group in both layouts; a thread's loads of a
  // round go out together
  const int ng = a.d >> 3;
  h16x8 xh[2], xl[2], wv[2];
  auto group_k = [&](int g0, int u) { return 8 * min(g0 + u * 256 + tid, ng - 1); };
  auto load_x = [&](int g0) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const h16_t* x = a.x.p + a.x.group_offset(r, group_k(g0, u));
      xh[u] = load_h16x8(x);
      xl[u] = a.x.planes == 2 ? load_h16x8(x + a.x.small_terms()) : zero_h16x8();
    }
  };
  auto load_w = [&](int g0, int t) {
#pragma unroll
    for (int u = 0; u < 2; ++u) wv[u] = load_h16x8(a.w_lm + packed_weight_offset(t, group_k(g0, u), a.d));
  };
  if (!SCORE) load_x(0);

  if (!sample_on) {                           // inert row
    if (tid == 0) {
      a.out_tokens[r] = a.pad;
      a.out_logprobs[r] = 0.f;
      if (a.out_sampled) a.out_sampled[r] = -1;
      if (!a.is_decode) a.finished[r] = 0;
    }
    return;
  }
  const bool capped = !SCORE && pos >= max_ctx_len - 1;
  int tok = capped ? a.eos : given ? forced : -1;
  const bool known = tok >= 0;                // uniform
  if (!SCORE && known) load_w(0, tok);
  // thread t takes tiles t, t + 256, ... (one 16-byte record each, eight loads in flight), merged in
  // ascending order; then a fixed binary tree over the threads
  Part p = {-INFINITY, 0.f, -INFINITY, 0x7FFFFFFF};
  for (int t0 = 0;;) {
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (t0 + u * 256 + tid < a.n_parts) {
        Part b = {q[u][0], q[u][1], q[u][2], __float_as_int(q[u][3])};
        p = part_merge(p, b);
      }
    t0 += 8 * 256;
    if (t0 >= a.n_parts) break;
    load_parts(t0);
  }
  for (int stride = 1; stride < 64; stride <<= 1) {
    const Part o = {__shfl_down(p.m, stride, WAVE), __shfl_down(p.s, stride, WAVE), __shfl_down(p.best, stride, WAVE),
                    __shfl_down(p.besti, stride, WAVE)};
    const Part n = part_merge(p, o);
    if ((tid & (2 * stride - 1)) == 0) p = n;
  }
  if ((tid & 63) == 0) sh[tid >> 6] = p;
  __syncthreads();
  p = part_merge(part_merge(sh[0], sh[1]), part_merge(sh[2], sh[3]));
  const float lse = p.m + logf(p.s);
  const int sampled = p.besti;
  if (!known) tok = sampled;
  if (tok < 0 || tok >= a.vocab) tok = a.eos;   // cannot happen with a non-empty vocabulary; keeps the read in bounds

  // logit of the emitted token: the same 16-bit operands as the LM-head tiles, fp32 accumulate
  const int dt = a.x.dtype;
  float acc = 0.f;
  for (int g0 = 0; g0 < ng; g0 += 2 * 256) {
    if (g0 || SCORE) load_x(g0);
    if (g0 || SCORE || !known) load_w(g0, tok);
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (g0 + u * 256 + tid < ng) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int sh = 16 * (e & 1);
          float xv = h16_to_f32((h16_t)((xh[u][e >> 1] >> sh) & 0xFFFFu), dt);
          if (a.x.planes == 2) xv += h16_to_f32((h16_t)((xl[u][e >> 1] >> sh) & 0xFFFFu), dt);
          acc += xv * h16_to_f32((h16_t)((wv[u][e >> 1] >> sh) & 0xFFFFu), dt);
        }
      }
  }
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) dsh[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (tid == 0) {
    float z = dsh[0] + dsh[1] + dsh[2] + dsh[3];
    float invt = temp > 0.f ? 1.f / temp : 1.f;
    a.out_logprobs[r] = z * invt - lse;
    if (SCORE) return;
    a.out_tokens[r] = tok;
    if (a.out_sampled) a.out_sampled[r] = sampled;
    uint8_t fin = (tok == a.eos) ? 1 : 0;
    if (a.is_decode) {
      a.finished[r] = fin;          // the row was live at entry
      a.ctx_lens[r] += 1;
    } else {
      a.finished[r] = fin;
    }
  }
}

}  // namespace

hipError_t sample_finalize(const FinalizeArgs& a, hipStream_t st) {
  if (a.score) hipLaunchKernelGGL(sample_finalize_kernel<true>, dim3(a.n_rows), dim3(256), 0, st, a);
  else hipLaunchKernelGGL(sample_finalize_kernel<false>, dim3(a.n_rows), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace rlx
