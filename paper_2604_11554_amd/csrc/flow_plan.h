// Which products of short calls take the form of gemm_flow.hip, and how it cuts them.  Plain host arithmetic on sizes.
#pragma once

namespace rlx {

constexpr int FLOW_WAVES = 4;
constexpr int FLOW_RT_MANY = 5;                      // row tiles per workgroup at most beside more than four token tiles (registers)

// ---- store form: row tiles per workgroup and planes of K ----
// A grid runs in `rounds` of one workgroup per compute unit, usually one (wide outputs take more), so the time is that of so many
// workgroups: what one takes in at 45 bytes/ns, its weights alone at 32 (or all of them at the card's 6.6 TB/s), its tiles' sums
// through LDS, and the planes that it and the kernel behind it write and read.  The constants (us) were fitted to a sweep of the
// 4B shape's products at 1 to 128 tokens; there the choice is within 4 % of the best one, or takes half the planes.  Against the
// skinny form, over nineteen products of 256 x 688 to 12 288 x 8192 and both formats: 0.53 to 1.04 of its time.
struct FlowPlan { int rt, splits; };   // row tiles of a workgroup, planes
constexpr int FLOW_RT[] = {2, 4, 5, 8};
inline FlowPlan flow_store_plan(int N, int K, int T, int max_splits, int n_units, int planes) {
  const int row_tiles = (N + 31) / 32 * 2, steps = (K / 16 + 1) / 2;
  const float all = (float)N * (float)K * 2.f / 6.6e6f;
  FlowPlan best = {2, 1};
  float best_us = 1e30f;
  for (int rt : FLOW_RT) {
    if (T > 64 && rt > FLOW_RT_MANY) continue;
    const int groups = (row_tiles + rt - 1) / rt;
    for (int s = 1; s <= max_splits; ++s) {
      const int per = (steps + s - 1) / s;
      if (s > 1 && ((s - 1) * per >= steps || per < FLOW_WAVES)) continue;   // no empty split, a step for every wave
      const float rounds = (float)((groups * s + n_units - 1) / n_units);
      const float kb = (float)((per + FLOW_WAVES - 1) / FLOW_WAVES * FLOW_WAVES) * 1.024f;   // of a row tile, or of a token tile and term
      float us = rounds * kb * ((float)rt + (float)(planes * T) / 16.f) / 45.f;
      const float weights = rounds * kb * (float)rt / 32.f;
      if (us < weights) us = weights;
      if (us < all) us = all;
      us += rounds * 0.12f * (float)(rt * ((T + 15) / 16)) + (float)s * (0.12f + 1e-6f * (float)T * (float)N);
      if (us < best_us) { best_us = us; best = {rt, s}; }
    }
  }
  return best;
}

// SwiGLU form (K whole): the fewest row tiles per workgroup that keep the grid within one workgroup per unit (4B shape, 64 tokens:
// 5 row tiles, 244 workgroups 25.4 us; 8, 152 30.9; 4, 304 38.4); 0: none does
constexpr int FLOW_SWIGLU_RT[] = {2, 4, 5, 6, 8};
inline int flow_swiglu_rt(int F, int T, int n_units) {
  for (int rt : FLOW_SWIGLU_RT)
    if ((F / 8 + rt - 1) / rt <= n_units) return T > 64 && rt > FLOW_RT_MANY ? 0 : rt;
  return 0;
}

// Stores of two terms: up to 96 tokens (at 97 to 128 the skinny form's two groups of 64 are as fast or faster).  Of 49 to 64 tokens,
// the skinny form's own tile, only the narrower ones: what this form saves there are planes of K, of which the skinny form needs
// n_units / (N / 128) to fill the device.  Where five or fewer do, the two are even (us, skinny -> this form, 64 tokens, N x K
// 6144 x 2560 11.4 -> 11.8, 6144 x 4096 15.4 -> 15.9, 7168 x 5120 19.3 -> 19.3, 9216 x 4096 21.6 -> 20.9); with more this one is
// faster (5120 x 2048 9.6 -> 8.8, 3072 x 2048 7.7 -> 7.3, 1536 x 1024 6.5 -> 4.5, 768 x 256 6.2 -> 3.9; 2560 x 9728 15.8 -> 14.7).
// And only where the activations stay in an XCD's 4 MB of L2, from where the workgroups read them again and again: N x K 8192 x
// 22016, 80 tokens (7.0 MB) 119 -> 134 us, 96 (8.5 MB) 117 -> 150, fp16 128 (5.6 MB) 96 -> 114; while 5120 x 13824, 96 tokens
// (5.3 MB) 51.8 -> 52.4, 80 (4.4 MB) 52.9 -> 41.6, 4096 x 12288, 96 (4.7 MB) 36.6 -> 33.9.
// planes: activations as two bf16 terms or one fp16 term.
inline bool flow_store_form(int N, int K, int T, int n_units, int planes) {
  if ((long)planes * T * K * 2 > 5L << 20) return false;
  if (planes == 1) return T <= 128;
  return T <= 48 || (T <= 64 ? n_units / ((N + 127) / 128) > 5 : T <= 96);
}

// ---- the norm of the rows inside the products that read them: every workgroup makes all rows ----
// What the kernels are built for: float4 slices of the rows per thread of 256, and rows of a token tile.
constexpr int FLOW_NORM_NV = 5, FLOW_NORM_ROWS = 16;
inline bool flow_norm_fits(int T, int K) { return T <= FLOW_NORM_ROWS && (long)T * (K / 4) <= FLOW_NORM_NV * 256L; }
// Where it pays.  A norm kernel before a product costs 3 to 4 us (its launch, a round trip for its row and another for the product's
// workgroups that wait for it); inside, a workgroup takes in the residual and the planes of the product before, which count
// as many times as there are planes, and adds up every row's squares: a row costs as much as 10 KB.  us a layer (two norms) saved in
// decode steps of two (d_model 256) or eight layers, bf16 / fp16, by the KB per product and the rows:
//   d_model 256    28 KB,  8 rows 1.4 / 1.9   35, 10  0.1 / 0.4   42, 12 -0.3 / 0.1   49, 14 -2.7 / -2.8   56, 16 -2.9 / -2.9
//           512    48,     4      2.2 / 2.7   72,  6  1.1 / 1.3   96,  8 -0.9 / -0.6  120, 10 -1.9 / -2.0
//          1024    56,     2      3.5 / 3.3   84,  3  2.3 / 3.2  112,  4 -0.1 / 0.6   140,  5 -0.9 / -2.1
//          1536    66,     2      2.9 / 4.4   99,  3  0.7 / 1.8
//    2048, 2560    80,     2      1.6 / 3.1, 2.0 / 4.6           2560 120, 3 -1.2      4096  48, 1 3.0 / 5.8
// and at full depth (36 layers, weights from memory), us a step, norm kernels / inside: 512, 8 rows 1102 / 1156, fp16 1109 / 1103;
// 1024, 3 rows 1316 / 1220, 4 1330 / 1304, fp16 1309 / 1276, 5 1359 / 1381, fp16 1341 / 1344; 1536, 3 rows 1632 / 1624; 2560, 2 rows
// 2246 / 2169.
// The line is 152 KB per product: what it takes saves something everywhere, or is even.
inline bool flow_norm_form(int T, int K, int planes_o, int planes_down) {
  const long kb = (long)T * K * 4 * (2 + planes_o + planes_down) / 1024;   // of both products of a layer
  return flow_norm_fits(T, K) && kb + 20L * T <= 305;
}

}  // namespace rlx
