// Which tiles a product of a long call takes (gemm_long.hip), and into how many planes K is cut.  Plain host arithmetic on sizes.
#pragma once

namespace rlx {

enum { LONG_512x128 = 0, LONG_128x128, LONG_512x64, LONG_160x128, LONG_192x128,   // weight rows x tokens of a workgroup
       LONG_320x128, LONG_320x256 };                                              // ... of LM heads of few rows
struct LongPlan { int form, splits; };

// us of so many workgroups, `per` stages each: one per unit, a last round that is not full being a little shorter ...
inline float long_alone_us(long workgroups, int n_units, int per, float start, float stage) {
  const long rounds = (workgroups + n_units - 1) / n_units;
  const float full = (float)(workgroups - (rounds - 1) * n_units) / (float)n_units;
  return (float)rounds * (start + stage * (float)per) - 0.1f * (1.f - full) * stage * (float)per;
}
// ... and of 128 x 128, two per unit, or one in a last round that has no more
inline float long_pairs_us(long workgroups, int n_units, int per) {
  const long full = workgroups / (2 * n_units), rest = workgroups % (2 * n_units);
  float us = (float)full * (3.5f + 0.79f * (float)per);
  if (rest) us += 3.5f + (rest <= n_units ? 0.464f : 0.79f) * (float)per;
  return us;
}

// 512 x 128 (eight waves, one workgroup per unit) has the better rate when the device is full many times over, 128 x 128
// (four waves, two workgroups per unit) an eighth of its step in size, 160 x 128 and 192 x 128 (four waves, one per unit, a wave
// all weight rows and 32 tokens) make one even round of 129 to 512 tokens where the others fill it and a half; what decides
// at a few hundred to a few thousand tokens is how well the workgroups fit the units.  The constants (us: start of a round, and
// per stage) were fitted to a sweep of the products of the two model shapes (N 2048..19456, K 2048..9728), 140..8192 tokens and
// 1 to 8 planes, where the choice is 0.1 % behind the best of the sweep in the mean and 4 % at worst (6 % in a second sweep at other
// token counts: N 5120, K 2048, 1700 tokens 83 us in 128 x 128, 88 in the chosen 512 x 128).  E.g. gate/up of 256
// tokens, N 19456, K 2560: 128 x 128 (304 workgroups) 65 us, 160 x 128 (244) 51; 1437 tokens, N 6144, K 2560: 128 x 128 in two
// planes 96 us, 512 x 128 in three 88; 8192 tokens, N 2560, K 9728: 128 x 128 692, 512 x 128 in two planes 629.
// `finest`: as many planes as there may be, in the form that is faster with them.
inline LongPlan long_plan(int N, int K, int T, int max_splits, int n_units, bool finest) {
  const int stages = (K / 16 + 1) / 2;
  LongPlan best = {LONG_512x128, 1};
  float best_us = 1e30f;
  for (int s = 1; s <= max_splits; ++s) {
    const int per = (stages + s - 1) / s;
    if (s > 1 && ((s - 1) * per >= stages || per < 8)) continue;   // no empty split, no split of a few stages
    if (finest) best_us = 1e30f;
    const long wg_t = (long)((T + 127) / 128) * s;
    const float planes_us = (float)(s - 1) * (float)T * (float)N * 0.94e-6f;
    auto take = [&](int form, float us) {
      us += planes_us;
      if (us < best_us) { best_us = us; best = {form, s}; }
    };
    auto alone = [&](int form, int rows, float start, float stage) {
      take(form, long_alone_us(wg_t * ((N + rows - 1) / rows), n_units, per, start, stage));
    };
    alone(LONG_512x128, 512, 5.0f, 1.29f);
    alone(LONG_160x128, 160, 3.8f, 0.67f);
    alone(LONG_192x128, 192, 3.2f, 0.785f);
    take(LONG_128x128, long_pairs_us(wg_t * ((N + 127) / 128), n_units, per));
  }
  return best;
}

// The LM head, whose epilogue makes the rounds longer where nothing runs beside them.  Up to LM_FEW_ROWS rows there are two forms
// more, 320 vocabulary rows by 128 or 256 tokens (eight waves, one workgroup per unit): they read the weights once for all rows and
// a wave's 160 ids are one part of the partials, but a workgroup takes two thirds of a 512 x 128 tile's time or more, so that what
// decides is how well the rounds fit the vocabulary.  us that a decode step takes longer than with the fastest, 512 x 128 / 128 x 128 /
// 320 x 128 / 320 x 256, K 2560 (one draw per row, no logits):
//   vocabulary        32 000              100 352              128 256              151 936
//      96 rows   55 /   0 /  23 /  43    0 /  27 /  40 /  71    0 /  18 /  28 /  60   73 /  26 /   0 /  30
//     128 rows   53 /   0 /  17 /  34    0 /  24 /  50 /  69    0 /  14 /  34 /  49   68 /   8 /   0 /  16
//     256 rows   33 /   0 /   1 /  60    0 /   5 /   1 /  55    0 /  20 /  62 /  38   50 /  35 /  18 /   0
// and K 2048, 151 936 ids, 96, 128, 256 rows:  67 /  14 /   0 /  22,  61 /   0 /   6 /   5,  45 /  23 /  18 /   0.
// The constants (us: start of a round, per stage, share of a last round's time that goes with its fill -- of 128 x 128, share that a round
// of one workgroup per unit takes --, share of a stage's that goes with the waves that have tokens) were fitted to 472 decode steps
// of two or three layers, 16 000 to 200 064 ids, K 256 to 4096, 65 to 256 rows.  In the mean the choice is 1.0 % of the LM head's time
// behind the best of the four, where the first two forms alone were 5.3 % and 320 rows at any vocabulary 43 %; where one of the first
// two is best it is 3 % behind at worst.  Past 256 rows those two are within 2 % of the others.
constexpr int LM_FEW_ROWS = 256;
inline int long_lmhead_form(int V, int K, int T, int n_units) {
  const int per = (K / 16 + 1) / 2;
  auto workgroups = [&](int rows, int tokens) { return (long)((T + tokens - 1) / tokens) * ((V + rows - 1) / rows); };
  if (T > LM_FEW_ROWS)
    return long_alone_us(workgroups(512, 128), n_units, per, 10.f, 1.4f) <= long_pairs_us(workgroups(128, 128), n_units, per)
               ? LONG_512x128 : LONG_128x128;
  int best = LONG_512x128;
  float best_us = 1e30f;
  // `wave`: tokens of a wave, `at_once`: workgroups of a round
  auto take = [&](int form, int rows, int tokens, int wave, int at_once, float start, float stage, float last, float empty) {
    const long w = workgroups(rows, tokens), full = w / at_once, rest = w % at_once;
    const float live = (float)((T + wave - 1) / wave * wave) / (float)((T + tokens - 1) / tokens * tokens);
    const float round = start + stage * (float)per * (1.f - empty * (1.f - live));
    float us = (float)full * round;
    if (rest) us += form != LONG_128x128 ? round * (1.f - last * (1.f - (float)rest / (float)at_once))
                                         : round * (rest <= n_units ? last : 1.f);   // one per unit is no slower by fill
    if (us < best_us) { best_us = us; best = form; }
  };
  take(LONG_512x128, 512, 128, 64, n_units, 28.5f, 1.46f, 0.30f, 0.43f);
  take(LONG_128x128, 128, 128, 64, 2 * n_units, 10.3f, 0.86f, 0.57f, 0.74f);
  take(LONG_320x128, 320, 128, 32, n_units, 16.7f, 1.09f, 0.31f, 0.52f);
  take(LONG_320x256, 320, 256, 64, n_units, 26.3f, 1.97f, 0.21f, 0.76f);
  return best;
}
// weight tiles (32 vocabulary rows each) of a part of an LM head's partials
inline int long_lmhead_part_tiles(int form) { return form == LONG_320x128 || form == LONG_320x256 ? 5 : 2; }

}  // namespace rlx
