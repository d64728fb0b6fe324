// Descriptor of the shared prompt prefixes of a decode batch: what it holds, and how the host fills it.  Plain host arithmetic, but
// for the sizes that the kernels use too.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

namespace rlx {

// int32 words (built on the host, read by the kernels):
//   [0] n_seqs it was built for, [1] n_tiles, [2] members per tile MS = min(16, SP_COLS / (Hq/Hkv)),
//   [3] 1 if the tiles' pages are copied without the streaming mark (shared_prefix_plain), [4..7] 0
//   per sequence (4 arrays of n_seqs): start_unit, tile0 (first tile of its subgroup), n_chunks, col0 (its first column)
//   per tile (arrays of max_tiles; groups of the longest chunks first): row (sequence whose block-table row lists the pages), kvh,
//   unit lo, unit hi,
//   then members [max_tiles][16] (-1 = none).  Tile of (subgroup, chunk c, kvh) = tile0 + c * Hkv + kvh.
constexpr int SP_HDR = 8;
constexpr int SP_MAX_CHUNKS = 4;
constexpr int SP_COLS = 32;          // columns of a prefix tile: two matrix-core column tiles of 16
constexpr int shared_prefix_members(int group) { return group > 0 && SP_COLS / group < 16 ? SP_COLS / group : 16; }
// a subgroup has at least two members wherever the groups have, and at most one more subgroup per group than
// members / 2: tiles = subgroups x chunks x Hkv fit with at least one chunk each
constexpr int shared_prefix_max_tiles(int n_seqs, int Hkv) { return n_seqs * Hkv; }
inline size_t shared_prefix_words(int n_seqs, int Hkv) {
  return (size_t)SP_HDR + 4 * (size_t)n_seqs + (size_t)shared_prefix_max_tiles(n_seqs, Hkv) * (4 + 16);
}
// The units of a tile as its kernel walks them, whatever the words hold: 0 <= lo <= hi, unit hi - 1 in a block-table row of max_blocks
// entries (and, lo being no further than that, block 2 lo is an index that does not overflow).
struct PrefixRange { int lo, hi; };
constexpr PrefixRange prefix_range(int lo, int hi, int max_blocks) {
  const int most = hi < max_blocks / 2 ? hi : max_blocks / 2, end = most > 0 ? most : 0;
  return {lo < 0 ? 0 : lo < end ? lo : end, end};
}

// Groups that share something: sequences b .. e - 1, `units` of 32 keys.  A group is a run of consecutive sequences with the same
// leader (the first of them); its shared units are the smallest shared page count of its members, halved.
struct PrefixGroup { int b, e, units, chunks, per; };   // chunks of `per` units each, the last one shorter
inline std::vector<PrefixGroup> shared_prefix_groups(int n_seqs, const int32_t* leader, const int32_t* shared_pages) {
  std::vector<PrefixGroup> groups;
  for (int b = 0; b < n_seqs;) {
    int e = b + 1;
    while (e < n_seqs && leader[e] == b && leader[b] == b) ++e;
    const int units = *std::min_element(shared_pages + b, shared_pages + e) / 2;
    if (e - b >= 2 && units > 0) groups.push_back({b, e, units, 1, units});
    b = e;
  }
  return groups;
}

// Cuts the groups into at most `most_chunks` chunks of at least eight units (256 keys).  most_tiles (0: no limit): the workgroups that
// run at once.  Chunks get longer, the same for all groups, while the tiles are more than that, because a workgroup's second
// tile starts from nothing; but no longer than twice what an even deal gives a workgroup: past that a long prefix among short ones
// is the time of the whole launch (its units one after the other in one workgroup per KV head, four in flight), and splitting
// it costs tiles that run beside it.  Where even one chunk per group is more tiles than workgroups the bound alone decides.
// us a layer, 32 query and 8 KV heads, eight members a group, one round of tiles at any price / this / always from eight units:
// 64 prefixes of 40 units and one of 937: 392 / 129 / 169; 63 and one: 388 / 129 / 161; 70 of 16 to 64 and two of 500: 234 / 99 / 131; 39
// of 20 and one of 400: 58 / 58 / 59; 32 of 16 to 64: 38 / 38 / 41; 65 of 40: 80 / 80 / 81; 128 of 16 to 64: 118 / 119 / 144; 96 pairs of 8
// units and one of 937: 369 / 197 / 198.
// A step at full depth (36 layers), us, one round of tiles at any price / this: pairs, 64 prefixes of 640 positions and one of 15 000
// 13 290 / 10 140; groups of four, 70 of 256 to 1024 and two of 8000 13 380 / 11 070; groups of eight, 32 of 517 to 2048 9 270 / 9 200.
inline void shared_prefix_cut(std::vector<PrefixGroup>& groups, int MS, int Hkv, int most_chunks, int most_tiles) {
  constexpr int LEAST = 8;
  auto subgroups = [&](const PrefixGroup& g) { return (int64_t)((g.e - g.b + MS - 1) / MS); };
  auto cut = [&](const PrefixGroup& g, int least) {
    return (int)std::min<int64_t>(((int64_t)g.units + least - 1) / least, most_chunks);
  };
  int least = LEAST;
  if (most_tiles > 0) {
    int64_t all = 0;
    for (const PrefixGroup& g : groups) all += subgroups(g) * Hkv * g.units;
    auto fits = [&](int l) {
      int64_t tiles = 0;
      for (const PrefixGroup& g : groups) tiles += subgroups(g) * Hkv * cut(g, l);
      return tiles <= most_tiles;
    };
    const int64_t even = (all + most_tiles - 1) / most_tiles;
    int bound = (int)std::min<int64_t>(std::max<int64_t>(2 * even, LEAST), 1 << 30);   // units are fewer than that
    while (least < bound) {                          // the shortest that fit, or the bound
      const int mid = least + (bound - least) / 2;
      if (fits(mid)) bound = mid;
      else least = mid + 1;
    }
  }
  for (PrefixGroup& g : groups) {
    g.chunks = cut(g, least);
    g.per = (g.units + g.chunks - 1) / g.chunks;
    g.chunks = (g.units + g.per - 1) / g.per;          // no empty chunk
  }
}

// Whether pages are copied without the streaming mark: where a group has more members than a tile holds, so that several tiles
// read its pages, and where the shared pages of all layers stay in the card's 256 MB memory-side cache from one step to the next, which
// the mark keeps them out of.  us a step, 4B shape at full depth (36 layers, 590 KB a unit and KV head), with the mark / without,
// prefixes of half to all of so many positions: groups of eight, 320: one 2779 / 2767, two 2991 / 2981, four (140 MB) 3384 / 3349,
// eight (283 MB) 4175 / 4175, fp16 3862 / 3915; 16 groups of two, 320 (566 MB) 3404 / 3468; four of eight, 1000 (440 MB) 3400 / 3467.
constexpr int64_t SP_PLAIN_BYTES = 160ll << 20;
inline int64_t shared_prefix_plain_units(int hd, int n_layers) { return SP_PLAIN_BYTES / ((int64_t)128 * hd * n_layers); }
inline bool shared_prefix_plain(const std::vector<PrefixGroup>& groups, int MS, int Hkv, int64_t plain_units) {
  int64_t units = 0;
  bool again = false;
  for (const PrefixGroup& g : groups) { units += (int64_t)g.units * Hkv; again |= g.e - g.b > MS; }
  return again || units <= plain_units;
}

// fills `words` (shared_prefix_words entries) from per-sequence group leaders and shared page counts.  Groups of one, groups that
// share less than one unit, and models whose 32 columns hold a single sequence get no tiles.
inline void shared_prefix_build(int n_seqs, int Hq, int Hkv, const int32_t* leader, const int32_t* shared_pages, int most_tiles,
                                int64_t plain_units, int32_t* words) {
  const int group = Hq / Hkv, MS = shared_prefix_members(group);
  const int max_tiles = shared_prefix_max_tiles(n_seqs, Hkv);
  const size_t n_words = shared_prefix_words(n_seqs, Hkv);
  for (size_t i = 0; i < n_words; ++i) words[i] = 0;
  int32_t* start_unit = words + SP_HDR;
  int32_t *tile0 = start_unit + n_seqs, *n_chunks = tile0 + n_seqs, *col0 = n_chunks + n_seqs;
  int32_t* t_row = col0 + n_seqs;
  int32_t *t_kvh = t_row + max_tiles, *t_lo = t_kvh + max_tiles, *t_hi = t_lo + max_tiles, *t_mem = t_hi + max_tiles;
  for (int i = 0; i < max_tiles * 16; ++i) t_mem[i] = -1;
  words[0] = n_seqs; words[2] = MS;
  if (MS < 2) return;
  std::vector<PrefixGroup> groups = shared_prefix_groups(n_seqs, leader, shared_pages);
  int64_t subgroups = 0;
  for (const PrefixGroup& g : groups) subgroups += (g.e - g.b + MS - 1) / MS;
  const int most_chunks = subgroups ? (int)std::min<int64_t>(max_tiles / (subgroups * Hkv), SP_MAX_CHUNKS) : 0;
  if (most_chunks < 1) return;
  shared_prefix_cut(groups, MS, Hkv, most_chunks, most_tiles);
  // the longest tiles first: a workgroup's second one comes from the other end of the list
  std::stable_sort(groups.begin(), groups.end(), [](const PrefixGroup& x, const PrefixGroup& y) { return x.per > y.per; });
  words[3] = shared_prefix_plain(groups, MS, Hkv, plain_units);
  int n_tiles = 0;
  for (const PrefixGroup& g : groups) {
    for (int sb = g.b; sb < g.e; sb += MS) {
      const int se = sb + MS < g.e ? sb + MS : g.e;
      for (int i = sb; i < se; ++i) {
        start_unit[i] = g.units; tile0[i] = n_tiles; n_chunks[i] = g.chunks; col0[i] = (i - sb) * group;
      }
      for (int c = 0; c < g.chunks; ++c)
        for (int h = 0; h < Hkv; ++h) {
          const int t = n_tiles + c * Hkv + h;
          t_row[t] = g.b; t_kvh[t] = h; t_lo[t] = c * g.per; t_hi[t] = std::min((c + 1) * g.per, g.units);
          for (int i = sb; i < se; ++i) t_mem[t * 16 + (i - sb)] = i;
        }
      n_tiles += g.chunks * Hkv;
    }
  }
  words[1] = n_tiles;
}

}  // namespace rlx
