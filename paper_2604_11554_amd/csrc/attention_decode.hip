// Decode attention over the paged 16-bit KV pool, load-balanced by key count.
//
// One new token per sequence; the 16 MFMA columns of a tile are the query heads of one KV head
// (group <= 16), so a KV page is read once for all heads of its group.  The work of a step is the
// sequence of 32-key units of all (sequence, KV head) pairs laid end to end; every WAVE takes a
// contiguous share of it, all shares within one unit of each other (the plan is built once per step,
// contexts being the same for every layer), on a grid that is exactly resident (two workgroups of four waves per
// compute unit).  A wave walks its share by itself, the next unit's pages on their way while it works on the current
// one, the next pair's queries copied into its part of LDS by the hardware; there is no barrier.  Where a (sequence, KV
// head) pair lies inside one share its output is final; elsewhere each part leaves (o, m, l) and a small second kernel
// merges the parts in share order (deterministic).
// (Shares in fours, merged by their workgroup where they were exactly one pair -- equal contexts, as many pairs as
// workgroups: 4B shape, eight layers, 64 sequences of 1024 keys each 1160 us against 1200, but 64 of 769 to 1525 keys 1253
// against 1243, dense_b64's steps 5.39 ms against 5.34, and steps of few keys got shares of two units in series.)
// (With a share per workgroup, its waves taking units in turn, the end of every pair cost a merge of the four waves
// through LDS, three barriers and a half-idle step.  4B shape, 256 sequences, one layer: 32 to 287 keys each 94 us then,
// 42 now; 144 keys each 51 and 35; 1024 keys each 182 and 172, 6.2 TB/s.  A lone sequence of 3000 keys: merge 19 us
// then, of 64 parts by one round trip per four, 5 now.)
//
// MoE policies (a.team) keep a share per WORKGROUP instead, its four waves taking the share's units in turn and merging
// their sums through LDS: another order of sums is not wrong, but it moves the last bits of the router's input, and a token
// at a near-tie of its eighth and ninth expert goes the other way.  30B-A3B shape, four layers, 128 sequences of 1530 keys:
// 1.41 ms a step with a share per wave, 1.39 to 1.43 with one per workgroup.
//
// Shared prompt prefixes (sequences of one sampling group list the same pages for their prompt): the descriptor
// `shared` names, per sequence, how many leading units are served by prefix tiles instead.  A prefix tile is
// (subgroup of up to 32 / group sequences, KV head, chunk of units): the 32 columns of its two MFMA column tiles
// are the query heads of all its member sequences, so the shared pages are read once per subgroup (the eight
// responses of a prompt at the 4B shape) instead of once per sequence; the per-sequence kernel starts after the
// shared units, and the merge kernel adds the prefix parts first.
#include <mutex>
#include <type_traits>

#include "attn_core.h"
#include "embed.h"
#include "lds_copy.h"
#include "rope.h"

namespace rlx {
namespace {

template <int HD>
struct PageRegs {
  h16x8 k0[HD / 32], k1[HD / 32], vf[HD / 16];
  bool ok0, ok1;
};

// Views into the shared-prefix descriptor (kernels.h); `on` is false when there is none or it was built for
// another batch size, and every index read from it is clamped by its user.
struct SharedView {
  bool on, plain;                                    // plain: pages are copied without the streaming mark
  int n_tiles, max_tiles;
  const int32_t *start_unit, *tile0, *n_chunks, *col0, *t_row, *t_kvh, *t_lo, *t_hi, *t_mem;
};
__device__ __forceinline__ SharedView shared_view(const int32_t* sp, int n_seqs, int Hkv) {
  SharedView v = {};
  if (sp == nullptr) return v;
  typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
  const i32x4 head = *reinterpret_cast<const i32x4*>(sp);     // at once: one round trip before anything else is read
  v.on = head[0] == n_seqs;
  if (!v.on) return v;
  v.max_tiles = shared_prefix_max_tiles(n_seqs, Hkv);
  v.n_tiles = min(max(head[1], 0), v.max_tiles);
  v.plain = head[3] != 0;
  const int32_t* p = sp + SP_HDR;
  v.start_unit = p; v.tile0 = p + n_seqs; v.n_chunks = p + 2 * n_seqs; v.col0 = p + 3 * n_seqs;
  p += 4 * (size_t)n_seqs;
  v.t_row = p; v.t_kvh = p + v.max_tiles; v.t_lo = p + 2 * (size_t)v.max_tiles; v.t_hi = p + 3 * (size_t)v.max_tiles;
  v.t_mem = p + 4 * (size_t)v.max_tiles;
  return v;
}
// units of sequence `seq` that prefix tiles serve: never all of them (its own kernel keeps at least one unit)
__device__ __forceinline__ int shared_units_of(const SharedView& v, int seq, int ctx) {
  return v.on ? min(max(v.start_unit[seq], 0), ctx / 32) : 0;
}

// Shares of two sizes: 0 .. H-1 take CA units each, the others CB = CA - 1 as long as there are units (plan header: CA,
// total, CB, H).
struct Shares {
  int CA, CB, H, U;
  __device__ __forceinline__ int start(int w) const { return w < H ? w * CA : H * CA + (w - H) * CB; }
  __device__ __forceinline__ int of_unit(int x) const { return x < H * CA ? x / CA : H + (x - H * CA) / max(CB, 1); }   // x < U
};
__device__ __forceinline__ Shares load_shares(const int32_t* hdr) { return Shares{hdr[0], hdr[2], hdr[3], hdr[1]}; }

// A run: up to 64 consecutive units of one (sequence, KV head) inside a share (64 units = one register window of the
// block table).  A segment -- the part of a pair that lies in the share -- is one or more runs; the online softmax state
// lives across the runs of a segment.  All fields are wave-uniform.
struct Run {
  int seq, kvh, ctx, np;     // np: units of the whole pair, counted from unit u0 of the sequence
  int u0;                    // units before this pair's first one (served by prefix tiles)
  int pb, pe;                // units [pb, pe) of the pair are this share's segment
  int lo, hi;                // units [lo, hi) of the pair are this run
  bool seg_start, seg_end, valid;
};

// Where a share starts, as the plan writes it (one 64-byte record, so that a share's first pages are two round trips away):
// sequence, KV head, ctx, u0 and np of its first pair, the share's first unit counted from that pair's, the share's units
// [u, u_end) on the line (none if u >= u_end), and the pages of its first units, two each, up to the segment's last one.
constexpr int SHARE_WORDS = ATTN_SHARE_WORDS, SHARE_BLOCKS = 8, SHARE_FIRST_UNITS = (SHARE_WORDS - SHARE_BLOCKS) / 2;
struct ShareStart {
  int seq, kvh, ctx, u0, np, pb, u, u_end;
  int32_t blocks[2 * SHARE_FIRST_UNITS];
  __device__ __forceinline__ int pe() const { return min(np, u_end - (u - pb)); }   // end of the first segment
};
__device__ __forceinline__ ShareStart load_share(const int32_t* recs, int w) {
  const int32_t* r = recs + (size_t)w * SHARE_WORDS;
  ShareStart s = {r[0], r[1], r[2], r[3], r[4], r[5], r[6], r[7], {}};
#pragma unroll
  for (int i = 0; i < 2 * SHARE_FIRST_UNITS; ++i) s.blocks[i] = r[SHARE_BLOCKS + i];
  return s;
}

// Walks the runs of a share: the per-sequence plan entries are held in a 64-lane register window.  The first run is known from
// the share's record; the window is requested with it and read when the walk goes on.
struct RunWalk {
  const AttnDecodeArgs& a;
  const SharedView sv;
  const int lane, u_end;
  int u, seq, seq0, rem_lo, rem_hi;                  // rem: rest of the current segment
  int32_t wpre, wctx, wst;
  Run seg;
  __device__ __forceinline__ RunWalk(const AttnDecodeArgs& args, int lane_, const ShareStart& s, Run& r)
      : a(args), sv(shared_view(args.shared, args.n_seqs, args.Hkv)), lane(lane_), u_end(s.u_end) {
    seg.seq = s.seq; seg.kvh = s.kvh; seg.ctx = s.ctx; seg.np = s.np; seg.u0 = s.u0;
    seg.pb = s.pb; seg.pe = s.pe();
    seg.valid = true;
    r = seg;
    r.lo = seg.pb; r.hi = min(seg.pe, seg.pb + 64);
    r.seg_start = true; r.seg_end = r.hi == seg.pe;
    rem_lo = r.hi; rem_hi = seg.pe;
    u = s.u - s.pb + seg.pe;
    seq = s.seq + (seg.pe == seg.np && seg.kvh == a.Hkv - 1 ? 1 : 0);
    slide();
  }
  __device__ __forceinline__ void slide() {
    seq0 = seq;
    wpre = a.unit_prefix[min(seq0 + lane, a.n_seqs)];
    wctx = a.ctx_lens[min(seq0 + lane, a.n_seqs - 1)];
    wst = shared_units_of(sv, min(seq0 + lane, a.n_seqs - 1), wctx);
  }
  __device__ __forceinline__ void next(Run& r) {
    if (rem_lo < rem_hi) {                           // the segment continues in another table window
      r = seg;
      r.lo = rem_lo; r.hi = min(rem_hi, rem_lo + 64);
      r.seg_start = false; r.seg_end = r.hi == rem_hi;
      rem_lo = r.hi;
      return;
    }
    r.valid = false;
    while (u < u_end && seq < a.n_seqs) {
      if (seq - seq0 > 62) slide();                  // rare: 63 sequences inside one share
      const int p0 = __builtin_amdgcn_readlane(wpre, seq - seq0);
      const int np = __builtin_amdgcn_readlane(wpre, seq - seq0 + 1) - p0;
      if (np == 0) { ++seq; continue; }              // inert sequence: no units
      const int base = a.Hkv * p0;
      const int kvh = (u - base) / np;
      if (kvh >= a.Hkv) return;                      // inconsistent plan: stop rather than index past the pool
      const int xs = base + kvh * np;                // first unit of this (sequence, KV head)
      seg.seq = seq; seg.kvh = kvh; seg.np = np;
      seg.ctx = __builtin_amdgcn_readlane(wctx, seq - seq0);
      seg.u0 = __builtin_amdgcn_readlane(wst, seq - seq0);
      seg.pb = u - xs; seg.pe = min(np, u_end - xs);
      seg.valid = true;
      r = seg;
      r.lo = seg.pb; r.hi = min(seg.pe, seg.pb + 64);
      r.seg_start = true; r.seg_end = r.hi == seg.pe;
      rem_lo = r.hi; rem_hi = seg.pe;
      u = xs + seg.pe;
      if (seg.pe == np && kvh == a.Hkv - 1) ++seq;
      return;
    }
  }
};

// block-table window of a run: lane holds the entries of blocks 2 (u0 + lo) + lane and + 64
__device__ __forceinline__ void load_window(const AttnDecodeArgs& a, const Run& r, int lane, int32_t& t0, int32_t& t1) {
  const int32_t* table = a.block_table + (size_t)r.seq * a.max_blocks;
  const int jb = 2 * (r.u0 + r.lo) + lane;
  const int j0 = min(jb, a.max_blocks - 1), j1 = min(jb + 64, a.max_blocks - 1);
  t0 = table[j0]; t1 = table[j1];                    // unconditional, clamped; masked below
  if (jb >= a.max_blocks) t0 = -1;
  if (jb + 64 >= a.max_blocks) t1 = -1;
}

// Page loads of unit i of run r, pages b0_ and b1_.  They are unconditional: a slot with no unit behind it
// (`live` false, i clamped into the run) reads one fixed row of the pool with every lane, which costs cache
// hits and no memory traffic.
template <int HD>
__device__ __forceinline__ void issue_pages(const AttnDecodeArgs& a, const Run& r, int32_t b0_, int32_t b1_, int i, bool live, int c16,
                                            int g, PageRegs<HD>& pr) {
  constexpr size_t page = (size_t)2 * 16 * HD;
  int64_t b0 = b0_, b1 = b1_;
  const bool has1 = (2 * (r.u0 + i) + 1) * 16 < r.ctx + 1;
  pr.ok0 = live && b0 >= 0 && b0 < a.n_blocks;
  pr.ok1 = live && has1 && b1 >= 0 && b1 < a.n_blocks;
  if (!pr.ok0) b0 = 0;                               // keep the loads in bounds; scores are masked
  if (!pr.ok1) b1 = b0;
  const h16_t* kp0 = a.pool_layer + ((size_t)b0 * a.Hkv + r.kvh) * page;
  const h16_t* kp1 = a.pool_layer + ((size_t)b1 * a.Hkv + r.kvh) * page;
  const h16_t* vp0 = kp0 + 16 * HD;
  const h16_t* vp1 = kp1 + 16 * HD;
  const int koff0 = pr.ok0 ? c16 * HD + 8 * g : 0, koff1 = pr.ok1 ? c16 * HD + 8 * g : 0;
  const int voff0 = pr.ok0 ? c16 * 16 + 4 * g : 0, voff1 = pr.ok1 ? c16 * 16 + 4 * g : 0;
#pragma unroll
  for (int ks = 0; ks < HD / 32; ++ks) {
    pr.k0[ks] = load_stream_16(kp0 + koff0 + 32 * ks);
    pr.k1[ks] = load_stream_16(kp1 + koff1 + 32 * ks);
  }
#pragma unroll
  for (int dt = 0; dt < HD / 16; ++dt)
    pr.vf[dt] = load_2x4_stream(vp0 + 256 * dt + voff0, vp1 + 256 * dt + voff1);
}

// The same with the pages taken from the run's table window t0/t1.
template <int HD>
__device__ __forceinline__ void issue_unit(const AttnDecodeArgs& a, const Run& r, int32_t t0, int32_t t1, int i, bool live, int c16,
                                           int g, PageRegs<HD>& pr) {
  const int rel = 2 * (i - r.lo);                    // uniform, 0 .. 126
  const int32_t sel = rel < 64 ? t0 : t1;
  issue_pages<HD>(a, r, __builtin_amdgcn_readlane(sel, rel & 63), __builtin_amdgcn_readlane(sel, (rel + 1) & 63), i, live, c16, g, pr);
}

// The end of a segment: final if it is a whole pair that no prefix precedes, else (o, m, l) for the merge kernel.  `share`:
// index of its share, `first`: it is the share's first segment.  Every lane of the wave calls it; a lane holds column
// c16, rows d = 16 dt + 4 g + {0..3}.
template <int HD, int PL, int FMT>
__device__ __forceinline__ void store_segment(const AttnDecodeArgs& a, const WaveState<HD, 1>& st, const Run& r, int share, bool first,
                                              int group, int c16, int g) {
  constexpr int PS = HD + 4;
  const bool col_ok = c16 < group, whole = r.pb == 0 && r.pe == r.np;
  if (whole && r.u0 == 0) {
    store_column<HD, 1, PL, FMT>(st, 0, a.o, r.seq, r.kvh * group + c16, g, col_ok);
  } else if (col_ok) {
    float* dst = whole ? a.seq_part + (((size_t)r.seq * a.Hkv + r.kvh) * group + c16) * PS
                       : a.part + ((size_t)(share * 2 + (first ? 0 : 1)) * group + c16) * PS;
#pragma unroll
    for (int dt = 0; dt < HD / 16; ++dt) *reinterpret_cast<f32x4*>(dst + 16 * dt + 4 * g) = st.o[0][dt];
    if (g == 0) { dst[HD] = st.m[0]; dst[HD + 1] = st.l[0]; }
  }
}

// A share per wave (dense policies).
template <int HD, int PL, int FMT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_decode_kernel(AttnDecodeArgs a) {
  constexpr int KS = HD / 32, NQ = PL * KS;
  // query fragments of the wave's current and next pair, MFMA operand order
  __shared__ u32x4 lds_q[4][2][NQ * WAVE];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15, g = lane >> 4;
  const int group = a.Hq / a.Hkv;
  const bool col_ok = c16 < group;
  const int w = wave * gridDim.x + blockIdx.x;       // few shares spread over the units
  if (w >= ATTN_SHARES_MAX) return;
  const ShareStart share = load_share(a.share_start, w);
  if (share.u >= share.u_end) return;                // uniform over the wave
  const float scale = rsqrtf((float)HD);
  Run cur, nxt;
  RunWalk walk(a, lane, share, cur);
  // The query fragments of a pair go straight into LDS, a whole run before they are read (the run generator looks one
  // run ahead anyway).  Columns past the group read some head's queries; their results are never stored.
  int qsel = 0;
  auto copy_queries = [&](const Run& r, int sel) {
    const int head = r.kvh * group + (col_ok ? c16 : 0);
    const uint32_t dst = lds_address(&lds_q[wave][sel][0]);
#pragma unroll
    for (int f = 0; f < NQ; ++f) {
      const int p = f / KS, ks = f % KS;
      copy_to_lds(a.q.p + p * a.q.plane + ((size_t)r.seq * a.Hq + head) * HD + 32 * ks + 8 * g, dst + f * 1024);
    }
  };
  auto qf = [&](int p, int, int ks) { return __builtin_bit_cast(h16x8, lds_q[wave][qsel][(p * KS + ks) * WAVE + lane]); };

  int32_t tb0, tb1, tbn0, tbn1;
  load_window(a, cur, lane, tb0, tb1);
  copy_queries(cur, 0);

  WaveState<HD, 1> st;
  PageRegs<HD> ra, rb;
  issue_pages<HD>(a, cur, share.blocks[0], share.blocks[1], cur.lo, true, c16, g, ra);
  __builtin_amdgcn_sched_barrier(0);                 // everything that the record names is on its way before the walk goes on
  bool first_seg = true, more = false, fresh = true;
  int k = cur.lo;
  auto look_ahead = [&]() {                          // the run after cur: its table window and, for a new pair, its queries
    walk.next(nxt);
    more = nxt.valid;
    if (!more) nxt = cur;                            // keeps the look-ahead loads in bounds
    load_window(a, nxt, lane, tbn0, tbn1);
    if (more && nxt.seg_start) copy_queries(nxt, qsel ^ 1);
  };
  look_ahead();
  st.reset();

  // One unit: the next one's pages (of this run or the first of the next) are requested into `next`, then the unit in
  // `now` is multiplied.  There is no branch around the loads, so the hardware counters let a step wait for its own
  // pages only.  Returns false after the wave's last unit.
  auto unit = [&](PageRegs<HD>& now, PageRegs<HD>& next) -> bool {
    const bool last = k + 1 == cur.hi;
    {
      Run rs = cur;
      if (last) rs = nxt;
      issue_unit<HD>(a, rs, last ? tbn0 : tb0, last ? tbn1 : tb1, last ? nxt.lo : k + 1, !last || more, c16, g, next);
    }
    // The first unit of a pair: its queries were requested before its pages, and loads return in order, so the queries are
    // in LDS once the first of the pages is in its registers, which this statement asks of the compiler.
    if (fresh) asm volatile("" : "+v"(now.k0[0])::"memory");
    fresh = false;
    asm volatile("" ::: "memory");                   // query fragments are re-read from LDS, not kept in registers
    __builtin_amdgcn_sched_barrier(0);               // the next unit's loads go out before this unit's math
    const int key0 = 32 * (cur.u0 + k), key_end = cur.ctx + 1;
    const int pos_col[1] = {cur.ctx};
    pair_step<HD, 1, PL, FMT>(st, now.k0, now.k1, now.vf, qf, key0, key0 + 16, now.ok0, now.ok1, key_end, pos_col,
                              now.ok0 && now.ok1 && key0 + 32 <= key_end, scale, g);
    if (!last) { ++k; return true; }
    if (cur.seg_end) {
      st.finish_denominators();
      store_segment<HD, PL, FMT>(a, st, cur, w, first_seg, group, c16, g);
      first_seg = false;
      st.reset();
    }
    if (!more) return false;
    if (nxt.seg_start) { qsel ^= 1; fresh = true; }
    cur = nxt; tb0 = tbn0; tb1 = tbn1; k = cur.lo;
    look_ahead();
    return true;
  };
  while (unit(ra, rb) && unit(rb, ra)) {}
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no copy may outlive the workgroup's LDS
}

// A share per workgroup (MoE policies): the four waves take the share's units in turn, and their sums of a segment are
// merged through LDS.
template <int HD, int PL, int FMT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_decode_team_kernel(AttnDecodeArgs a) {
  constexpr int DT = HD / 16, KS = HD / 32;
  __shared__ f32x4 lds_o[2 * DT * WAVE];
  __shared__ float lds_ml[2 * 2 * WAVE];
  __shared__ u32x4 lds_q[PL * KS * WAVE];            // query fragments of the current segment, MFMA operand order

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15, g = lane >> 4;
  const int group = a.Hq / a.Hkv;
  const bool col_ok = c16 < group;
  const int w = blockIdx.x;
  const ShareStart share = load_share(a.share_start, w);
  if (share.u >= share.u_end) return;                // uniform over the workgroup
  const float scale = rsqrtf((float)HD);
  Run cur, nxt;
  RunWalk walk(a, lane, share, cur);
  // The waves share the fetch of a segment's query fragments; they stay in LDS (registers hold two units of pages).
  // The fragments of the next run's pair are requested a whole run ahead (the run generator looks one run ahead
  // anyway) and only written to LDS at the switch, so that a new segment does not begin with a round trip.
  constexpr int QPW = (PL * KS + 3) / 4;             // fragments fetched by each wave
  auto fetch_queries = [&](const Run& r, u32x4 (&q)[QPW]) {
    const int head = r.kvh * group + (col_ok ? c16 : 0);
#pragma unroll
    for (int i = 0; i < QPW; ++i) {
      const int f = min(wave + 4 * i, PL * KS - 1);  // a slot without a fragment repeats the last one; never written
      const int p = f / KS, ks = f % KS;
      q[i] = *reinterpret_cast<const u32x4*>(a.q.p + p * a.q.plane + ((size_t)r.seq * a.Hq + head) * HD + 32 * ks + 8 * g);
    }
  };
  auto put_queries = [&](const u32x4 (&q)[QPW]) {
    const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < QPW; ++i)
      if (wave + 4 * i < PL * KS) lds_q[(wave + 4 * i) * WAVE + lane] = col_ok ? q[i] : z;
  };
  auto qf = [&](int p, int, int ks) { return __builtin_bit_cast(h16x8, lds_q[(p * KS + ks) * WAVE + lane]); };

  int32_t tb0, tb1, tbn0, tbn1;
  load_window(a, cur, lane, tb0, tb1);
  u32x4 qpre[QPW];
  fetch_queries(cur, qpre);
  WaveState<HD, 1> st;
  PageRegs<HD> ra, rb;
  {
    int32_t b0 = share.blocks[0], b1 = share.blocks[1];
#pragma unroll
    for (int i = 1; i < 4; ++i)
      if (wave == i) { b0 = share.blocks[2 * i]; b1 = share.blocks[2 * i + 1]; }
    issue_pages<HD>(a, cur, b0, b1, min(cur.lo + wave, cur.hi - 1), cur.lo + wave < cur.hi, c16, g, ra);
  }
  __builtin_amdgcn_sched_barrier(0);                 // everything that the record names is on its way before the walk goes on
  put_queries(qpre);
  __syncthreads();

  bool first_seg = true;

  for (;;) {                                         // one run per iteration; uniform
    walk.next(nxt);
    const bool more = nxt.valid;
    if (!more) nxt = cur;                            // keeps the look-ahead loads below in bounds
    load_window(a, nxt, lane, tbn0, tbn1);
    fetch_queries(nxt, qpre);                        // unconditional, like every load of this loop
    if (cur.seg_start) st.reset();
    const int key_end = cur.ctx + 1;
    const int pos_col[1] = {cur.ctx};
    auto step = [&](int i, const PageRegs<HD>& pr, bool valid) {
      const int key0 = 32 * (cur.u0 + i);
      const bool ok0 = pr.ok0 && valid, ok1 = pr.ok1 && valid;
      pair_step<HD, 1, PL, FMT>(st, pr.k0, pr.k1, pr.vf, qf, key0, key0 + 16, ok0, ok1, key_end, pos_col,
                                ok0 && ok1 && key0 + 32 <= key_end, scale, g);
    };

    // Two register sets alternate: while one unit is multiplied the next one's pages are in flight.  The loop
    // body has no branch around a load (a unit index past the wave's last one is clamped and its step masked),
    // so the hardware counters let each step wait for its own pages only.  The slot after the wave's last unit
    // fetches its first unit of the next run, so the stream does not drain between runs.
    const int first = cur.lo + wave;
    const int n_my = first < cur.hi ? (cur.hi - first + 3) / 4 : 0;
    const int last = first + 4 * (n_my - 1);
    const int nfirst = min(nxt.lo + wave, nxt.hi - 1);
    const bool nlive = more && nxt.lo + wave < nxt.hi;
    for (int k = 0; k < n_my; k += 2) {
      const int i = first + 4 * k;
      issue_unit<HD>(a, cur, tb0, tb1, min(i + 4, last), i + 4 <= last, c16, g, rb);
      asm volatile("" ::: "memory");                 // query fragments are re-read from LDS, not kept in registers
      __builtin_amdgcn_sched_barrier(0);             // the next unit's loads go out before this unit's math
      step(i, ra, true);
      {
        const bool beyond = i + 8 > last;
        Run rs = cur;
        if (beyond) rs = nxt;
        issue_unit<HD>(a, rs, beyond ? tbn0 : tb0, beyond ? tbn1 : tb1, beyond ? nfirst : i + 8, !beyond || nlive, c16, g, ra);
      }
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      step(i + 4, rb, k + 1 < n_my);
    }
    if (n_my == 0) issue_unit<HD>(a, nxt, tbn0, tbn1, nfirst, nlive, c16, g, ra);   // this wave had no unit in the run

    if (cur.seg_end) {
      st.finish_denominators();
      merge_waves<HD, 1>(st, lds_o, lds_ml, wave, lane);
      if (wave == 0) store_segment<HD, PL, FMT>(a, st, cur, w, first_seg, group, c16, g);
      first_seg = false;
    }
    if (!more) break;
    if (nxt.seg_start) put_queries(qpre);            // every wave is past the merge: the old fragments are dead
    __syncthreads();                                 // new fragments visible; wave 0 is done with the merge buffers
    cur = nxt; tb0 = tbn0; tb1 = tbn1;
  }
}

// Prefix tiles: the workgroups walk the descriptor's tiles (tile_of).  The NCT x 16 columns are (member, head of the KV
// head's group); every key of the tile's units is visible to every member (the pages are full and shared).
// The four waves take units round-robin and are merged through LDS; (o, m, l) of all columns go to pre_part.  The
// query fragments of a tile sit in LDS (with two column tiles they would take half the register file).
// What bounds it: latency.  A wave has two to four units of a tile, and without registers for a second set of pages it waited for
// every one of them from the block table on.  The hardware now copies a unit's pages into the wave's part of LDS while the wave works
// on the one before, whose fragments are in registers by then (chunks permuted as in prefill attention: no bank conflicts); a tile's
// description, members and block-table entries are requested a tile ahead, and its queries behind its first pages.  Pages that one
// tile alone reads are copied with the streaming mark, but for few of them (shared_prefix_plain); tiles are as many as there are
// workgroups where chunks can be longer instead.
// us a layer of the 4B shape, before / copies / longest prefixes first / one round of tiles / streaming mark / longest tiles first:
// 32 groups of eight with prompts of 517 to 2048 positions 50.6 / 48.3 / 47.1 / 45.8 / 41.4 / 38.7 (168 MB, 4.3 TB/s); fp16, 32 of
// four, 400 to 1500, 38 / 35 / 34 / 32 / 29 / -; 16 groups of sixteen, whose pages two tiles read, 42 / - / - / - / 34 / -.  Short
// prompts (200 to 600) 21 before and now: the start, four round trips from the header to the pages, and the merge.
template <int HD, int NCT, int PL>
struct PrefixLds {
  static constexpr int UNIT = 4 * 16 * HD;           // elements of two pages of a KV head
  static constexpr int Q_BYTES = PL * NCT * (HD / 32) * WAVE * 16, PAGES_BYTES = 4 * UNIT * 2;
  static constexpr int O_BYTES = 2 * NCT * (HD / 16) * WAVE * 16, ML_BYTES = 2 * NCT * 2 * WAVE * 4;   // of the merge, over the pages
  static constexpr int BYTES = Q_BYTES + PAGES_BYTES;
  static_assert(O_BYTES + ML_BYTES <= PAGES_BYTES && BYTES <= 80 * 1024, "two workgroups per unit");
};
template <int HD, int PL, int FMT, int NCT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_decode_prefix_kernel(AttnDecodeArgs a) {
  constexpr int DT = HD / 16, KS = HD / 32, PS = HD + 4, NQ = PL * NCT * KS, RCH = HD / 8;
  constexpr int PAGE = 2 * 16 * HD, COPIES = PAGE * 2 / 1024;   // elements of a page, 1 KB copies of one
  typedef PrefixLds<HD, NCT, PL> L;
  extern __shared__ __align__(16) unsigned char prefix_lds[];
  u32x4* lds_q = reinterpret_cast<u32x4*>(prefix_lds);          // fragment (p, c, ks) at ((p * NCT + c) * KS + ks) * 64 + lane
  const SharedView sv = shared_view(a.shared, a.n_seqs, a.Hkv);
  if (!sv.on || (int)blockIdx.x >= sv.n_tiles) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15, g = lane >> 4;
  const int group = a.Hq / a.Hkv;
  const float scale = rsqrtf((float)HD);
  h16_t* my_pages = reinterpret_cast<h16_t*>(prefix_lds + L::Q_BYTES) + wave * L::UNIT;
  f32x4* lds_o = reinterpret_cast<f32x4*>(prefix_lds + L::Q_BYTES);
  float* lds_ml = reinterpret_cast<float*>(prefix_lds + L::Q_BYTES + L::O_BYTES);
  const uint32_t pages_at = lds_address(my_pages);

  // ---- what the tiles are ----
  struct Tile { int row, kvh, lo, hi, mem[NCT]; };   // all but the members uniform; mem: sequence of the lane's column, or out of range
  auto load_tile = [&](int t) {                      // requested, to be settled by `tile`
    Tile d;
    d.row = sv.t_row[t]; d.kvh = sv.t_kvh[t]; d.lo = sv.t_lo[t]; d.hi = sv.t_hi[t];
#pragma unroll
    for (int c = 0; c < NCT; ++c) {
      const int mi = (16 * c + c16) / group;
      d.mem[c] = sv.t_mem[(size_t)t * 16 + min(mi, 15)];
      if (mi > 15) d.mem[c] = -1;
    }
    return d;
  };
  auto tile = [&](Tile d) {
    d.row = min(max(__builtin_amdgcn_readfirstlane(d.row), 0), a.n_seqs - 1);
    d.kvh = min(max(__builtin_amdgcn_readfirstlane(d.kvh), 0), a.Hkv - 1);
    const PrefixRange r = prefix_range(__builtin_amdgcn_readfirstlane(d.lo), __builtin_amdgcn_readfirstlane(d.hi), a.max_blocks);
    d.lo = r.lo; d.hi = r.hi;
    return d;
  };
  // entries of the 32 units from unit `first` on: lane i holds block 2 first + i
  auto load_window = [&](const Tile& d, int first) {
    return a.block_table[(size_t)d.row * a.max_blocks + min(2 * first + lane, a.max_blocks - 1)];
  };

  // ---- copies of a unit: chunk (16 bytes) i * 64 + lane of a page comes from byte offset ... of it ----
  uint32_t k_off[COPIES / 2], v_off;                 // K rows' chunks permuted; V^T, 16 features at a time: the first chunks
#pragma unroll                                       // (tokens 0..7) of their rows, then the second
  for (int i = 0; i < COPIES / 2; ++i) {
    const int chunk = 64 * i + lane, row = chunk / RCH;
    k_off[i] = (uint32_t)(row * RCH + ((chunk % RCH) ^ (RCH == 16 ? row : (row >> 1) & 7))) * 16;
  }
  v_off = (uint32_t)(16 * RCH + ((lane >> 5) * 16 + (lane & 15)) * 2 + ((lane >> 4) & 1)) * 16;
  bool ok0 = false, ok1 = false;                     // of the unit in the wave's part of LDS
  auto copy_unit = [&](const Tile& d, int32_t window, int rel) {   // rel: unit counted from the window's first
    const int64_t n0 = __builtin_amdgcn_readlane(window, 2 * rel), n1 = __builtin_amdgcn_readlane(window, 2 * rel + 1);
    ok0 = n0 >= 0 && n0 < a.n_blocks;
    ok1 = n1 >= 0 && n1 < a.n_blocks;
    const int64_t b0 = ok0 ? n0 : 0, b1 = ok1 ? n1 : b0;   // keep the copies in bounds; scores are masked
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const unsigned char* page = reinterpret_cast<const unsigned char*>(a.pool_layer + ((size_t)(half ? b1 : b0) * a.Hkv + d.kvh) * PAGE);
      const uint32_t dst = pages_at + half * PAGE * 2;
      auto copy = [&](auto plain) {
        auto one = [&](const unsigned char* p, uint32_t off, uint32_t to) {
          if constexpr (decltype(plain)::value) copy_to_lds(p, off, to);
          else copy_to_lds_stream(p, off, to);
        };
#pragma unroll
        for (int i = 0; i < COPIES / 2; ++i) one(page, k_off[i], dst + i * 1024);
#pragma unroll
        for (int i = 0; i < COPIES / 2; ++i) one(page + i * 1024, v_off, dst + (COPIES / 2 + i) * 1024);
      };
      if (sv.plain) copy(std::true_type());
      else copy(std::false_type());
    }
  };

  // tiles of a workgroup: the list comes longest first and is walked to and fro, so that who begins with a long tile goes on
  // with a short one
  auto tile_of = [&](int k) { return k * (int)gridDim.x + (k & 1 ? (int)gridDim.x - 1 - (int)blockIdx.x : (int)blockIdx.x); };
  Tile d = tile(load_tile(blockIdx.x));
  int32_t window = load_window(d, d.lo);
  for (int k = 0; tile_of(k) < sv.n_tiles; ++k) {
    const int t = tile_of(k);
    int wlo = d.lo;                                  // first unit of the window
    if (d.lo + wave < d.hi) copy_unit(d, window, wave);
    // the waves share the fetch of the tile's query fragments
#pragma unroll
    for (int i = 0; i < (NQ + 3) / 4; ++i) {
      const int f = wave + 4 * i;
      if (f < NQ) {
        const int p = f / (NCT * KS), c = (f / KS) % NCT, ks = f % KS;
        int mem = d.mem[0];
#pragma unroll
        for (int cc = 1; cc < NCT; ++cc) mem = c == cc ? d.mem[cc] : mem;
        const bool col_ok = mem >= 0 && mem < a.n_seqs;
        const int head = d.kvh * group + (16 * c + c16) % group;
        u32x4 q = {0u, 0u, 0u, 0u};
        if (col_ok)
          q = *reinterpret_cast<const u32x4*>(a.q.p + p * a.q.plane + ((size_t)mem * a.Hq + head) * HD + 32 * ks + 8 * g);
        lds_q[f * WAVE + lane] = q;
      }
    }
    const Tile next = load_tile(min(tile_of(k + 1), sv.n_tiles - 1));
    __syncthreads();
    auto qf = [&](int p, int c, int ks) {
      return __builtin_bit_cast(h16x8, lds_q[((p * NCT + c) * KS + ks) * WAVE + lane]);
    };
    WaveState<HD, NCT> st;
    st.reset();
    int pos_col[NCT];
#pragma unroll
    for (int c = 0; c < NCT; ++c) pos_col[c] = 0x7FFFFFFF;
    for (int i = d.lo + wave; i < d.hi; i += 4) {    // 2 i + 1 < max_blocks by the clamp of hi
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the unit's pages are in LDS
      h16x8 k0[KS], k1[KS], vf[DT];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int off = c16 * HD + ((4 * ks + g) ^ (RCH == 16 ? c16 : (c16 >> 1) & 7)) * 8;
        k0[ks] = load_h16x8(my_pages + off);
        k1[ks] = load_h16x8(my_pages + PAGE + off);
      }
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const int off = 16 * HD + dt * 256 + (g >> 1) * 128 + c16 * 8 + (g & 1) * 4;
        vf[dt] = load_2x4(my_pages + off, my_pages + PAGE + off);
      }
      const bool o0 = ok0, o1 = ok1;
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // ... and in registers: the next one's may overwrite them
      if (i + 4 < d.hi) {
        if (i + 4 >= wlo + 32) { wlo += 32; window = load_window(d, wlo); }
        copy_unit(d, window, i + 4 - wlo);
      }
      __builtin_amdgcn_sched_barrier(0);
      pair_step<HD, NCT, PL, FMT>(st, k0, k1, vf, qf, 32 * i, 32 * i + 16, o0, o1, 0x7FFFFFFF, pos_col, o0 && o1, scale, g);
    }
    d = tile(next);
    window = load_window(d, d.lo);
    st.finish_denominators();
    __syncthreads();                                   // the pages' place is the merge's now
    merge_waves<HD, NCT>(st, lds_o, lds_ml, wave, lane);
    if (wave == 0) {
#pragma unroll
      for (int c = 0; c < NCT; ++c) {
        float* dst = a.pre_part + ((size_t)t * SP_COLS + 16 * c + c16) * PS;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) *reinterpret_cast<f32x4*>(dst + 16 * dt + 4 * g) = st.o[c][dt];
        if (g == 0) { dst[HD] = st.m[c]; dst[HD + 1] = st.l[c]; }
      }
    }
    __syncthreads();                                   // the merge buffers and the fragments are free for the next tile
  }
}

// One workgroup per (sequence, KV head): inert rows are zeroed; a pair that one share covered and no prefix precedes is
// already final; otherwise the parts are merged: prefix chunks in key order, then the pair's own part (one share) or
// parts (share order).  A thread owns eight features of a head; GROUPS threads share a slice and take a contiguous run of
// the parts each, a round trip per MERGE_BATCH of them, the first one the prefix chunks too; their results are merged in
// order through LDS.
//  - Shares per workgroup (MoE): one thread per slice, which keeps the sum in one run.
//  - Fewer than MERGE_MANY pairs: four.  The parts of the few pairs are many (a long context is dozens).
//  - More: two.  Most pairs have a handful of parts, and waves that find nothing to do cost too (2048 pairs, four instead
//    of one: 9.5 -> 12.7 us), but a sequence far longer than the others has hundreds.  4B shape, eight layers, 63 sequences
//    of 100 keys and one of 30 000 (198 parts): 1328 us with one thread per slice, 1195 with two, 1145 with four;
//    dense_b64's steps 5.36, 5.35 and 5.37 ms; 256 sequences in groups of eight 9.26, 9.24 and 9.25 ms.
constexpr int MERGE_GROUPS_MAX = 4, MERGE_BATCH = 8, MERGE_MANY = 512;
constexpr int MERGE_AT_ONCE = MERGE_GROUPS_MAX * MERGE_BATCH;
template <int HD, int GROUPS>
__global__ __launch_bounds__(256 * GROUPS) void attn_decode_merge_kernel(AttnDecodeArgs a) {
  constexpr int PS = HD + 4, PB = MERGE_BATCH;
  extern __shared__ __align__(16) float merge_lds[];   // [GROUPS - 1][slices][10]
  const int seq = blockIdx.x / a.Hkv, kvh = blockIdx.x % a.Hkv;
  const int group = a.Hq / a.Hkv, PL = a.o.planes;
  const int np = a.unit_prefix[seq + 1] - a.unit_prefix[seq];
  const Shares sh = load_shares(a.plan_hdr);
  const int xs = a.Hkv * a.unit_prefix[seq] + kvh * np;
  const int w_first = np ? sh.of_unit(xs) : 0, w_last = np ? sh.of_unit(xs + np - 1) : 0;
  const SharedView sv = shared_view(a.shared, a.n_seqs, a.Hkv);
  const int su = np ? shared_units_of(sv, seq, a.ctx_lens[seq]) : 0;
  if (np && w_first == w_last && su == 0) return;      // uniform over the workgroup
  int n_chunks = 0, tile0 = 0, col0 = 0;
  if (su > 0) {
    n_chunks = min(max(sv.n_chunks[seq], 0), SP_MAX_CHUNKS);
    tile0 = max(sv.tile0[seq], 0);
    col0 = min(max(sv.col0[seq], 0), SP_COLS - group);
  }
  const int slices = group * HD / 8;
  const int per_group = (int)blockDim.x / GROUPS;                           // at least `slices`, whole waves
  const int part_group = (int)threadIdx.x / per_group, uu = (int)threadIdx.x % per_group;
  const bool mine = uu < slices;
  const int us = mine ? uu : 0;
  const int j = us / (HD / 8), d0 = (us % (HD / 8)) * 8;
  float m = -INFINITY, l = 0.f;
  float o[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = 0.f;
  // a part of the pair, or (`other`) what comes from the other kernel's share of its keys: prefix chunks and the rest of a
  // pair that they precede (weighted_sum: the roundings of a few features differ between the two)
  auto add = [&](const f32x4& va, const f32x4& vb, float ms, float ls, bool other) {
    if (ms == -INFINITY) return;
    const float mn = fmaxf(m, ms);
    const float aa = state_weight(m, mn), ab = state_weight(ms, mn);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool swap = other && e == 0;
      o[e] = swap ? weighted_sum(va[e], ab, o[e], aa) : weighted_sum(o[e], aa, va[e], ab);
      o[4 + e] = swap ? weighted_sum(vb[e], ab, o[4 + e], aa) : weighted_sum(o[4 + e], aa, vb[e], ab);
    }
    l = other ? weighted_sum(ls, ab, l, aa) : weighted_sum(l, aa, ls, ab);
    m = mn;
  };
  auto add_at = [&](const float* p) {
    add(*reinterpret_cast<const f32x4*>(p + d0), *reinterpret_cast<const f32x4*>(p + d0 + 4), p[HD], p[HD + 1], true);
  };
  const int n_parts = np ? w_last - w_first + 1 : 0;
  if (part_group == 0 && n_chunks > 0) {
    f32x4 va[SP_MAX_CHUNKS], vb[SP_MAX_CHUNKS];
    float ms[SP_MAX_CHUNKS], ls[SP_MAX_CHUNKS];
#pragma unroll
    for (int c = 0; c < SP_MAX_CHUNKS; ++c) {          // loads first (clamped), merges after
      const int t = min(tile0 + min(c, n_chunks - 1) * a.Hkv + kvh, sv.max_tiles - 1);
      const float* p = a.pre_part + ((size_t)t * SP_COLS + col0 + j) * PS;
      va[c] = *reinterpret_cast<const f32x4*>(p + d0);
      vb[c] = *reinterpret_cast<const f32x4*>(p + d0 + 4);
      ms[c] = p[HD]; ls[c] = p[HD + 1];
    }
#pragma unroll
    for (int c = 0; c < SP_MAX_CHUNKS; ++c)
      if (c < n_chunks) add(va[c], vb[c], ms[c], ls[c], true);
  }
  if (n_parts == 1) {
    if (part_group == 0) add_at(a.seq_part + (((size_t)seq * a.Hkv + kvh) * group + j) * PS);
  } else {
    const int slot0 = xs <= sh.start(w_first) ? 0 : 1;
    // few parts stay with the first group: nothing to gain from dealing them out
    const int each = n_parts <= PB ? n_parts : (n_parts + GROUPS - 1) / GROUPS;
    const int p_b = min(n_parts, part_group * each), p_e = min(n_parts, p_b + each);
    for (int w0 = w_first + p_b; w0 < w_first + p_e; w0 += PB) {
      f32x4 va[PB], vb[PB];
      float ms[PB], ls[PB];
#pragma unroll
      for (int q = 0; q < PB; ++q) {                   // loads first (clamped), merges after
        const int wc = min(w0 + q, w_last);
        const int slot = wc == w_first ? slot0 : 0;    // first segment of its share or not
        const float* p = a.part + ((size_t)(wc * 2 + slot) * group + j) * PS;
        va[q] = *reinterpret_cast<const f32x4*>(p + d0);
        vb[q] = *reinterpret_cast<const f32x4*>(p + d0 + 4);
        ms[q] = p[HD]; ls[q] = p[HD + 1];
      }
#pragma unroll
      for (int q = 0; q < PB; ++q)
        if (w0 + q < w_first + p_e) add(va[q], vb[q], ms[q], ls[q], false);
    }
    if (GROUPS > 1 && n_parts > PB) {                  // uniform over the workgroup
      float* mine_lds = merge_lds + ((size_t)(part_group - 1) * slices + us) * 10;
      if (part_group > 0 && mine) {
#pragma unroll
        for (int e = 0; e < 8; ++e) mine_lds[e] = o[e];
        mine_lds[8] = m; mine_lds[9] = l;
      }
      __syncthreads();
      if (part_group == 0 && mine)
        for (int q = 0; q < GROUPS - 1; ++q) {
          const float* p = merge_lds + ((size_t)q * slices + us) * 10;
          add(f32x4{p[0], p[1], p[2], p[3]}, f32x4{p[4], p[5], p[6], p[7]}, p[8], p[9], false);
        }
    }
  }
  if (part_group > 0 || !mine) return;
  h16_t hi[8], lo[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) split_h16(l > 0.f ? o[e] / l : 0.f, hi[e], lo[e], a.o.dtype);
  h16_t* dst = a.o.p + a.o.group_offset(seq, (kvh * group + j) * HD + d0);
  u32x4 pk = {(uint32_t)hi[0] | ((uint32_t)hi[1] << 16), (uint32_t)hi[2] | ((uint32_t)hi[3] << 16),
              (uint32_t)hi[4] | ((uint32_t)hi[5] << 16), (uint32_t)hi[6] | ((uint32_t)hi[7] << 16)};
  *reinterpret_cast<u32x4*>(dst) = pk;
  if (PL == 2) {
    u32x4 pk2 = {(uint32_t)lo[0] | ((uint32_t)lo[1] << 16), (uint32_t)lo[2] | ((uint32_t)lo[3] << 16),
                 (uint32_t)lo[4] | ((uint32_t)lo[5] << 16), (uint32_t)lo[6] | ((uint32_t)lo[7] << 16)};
    *reinterpret_cast<u32x4*>(dst + a.o.small_terms()) = pk2;
  }
}

// The start of a decode step, one launch of n_seqs + 1 workgroups.  Workgroup 1 + i: metadata of row i, the rotary factors of
// its new position (the same for every layer, so they are computed once per step and not per layer) and its token's embedding.
// Workgroup 0, the plan of the step's attention: exclusive prefix of the per-sequence unit counts, the two share sizes, and
// where each share starts.
__global__ __launch_bounds__(1024) void decode_begin_kernel(DecodeBeginArgs b) {
  const int n_seqs = b.n_seqs, Hkv = b.Hkv;
  const int32_t* ctx = b.ctx_lens;
  if (blockIdx.x > 0) {
    const int i = blockIdx.x - 1, pos = ctx[i], half = b.head_dim / 2;
    embed_row(b.embed, b.vocab, b.d_model, b.tokens[i], nullptr, b.h + (size_t)i * b.d_model, b.dtype);
    for (int j = threadIdx.x; j < half; j += blockDim.x) {
      float c, s;
      rope_cos_sin(pos, b.inv_freq, true, j, c, s);
      b.meta.rope_cs[(size_t)i * half + j] = float2{c, s};
    }
    if (threadIdx.x != 0) return;
    const uint8_t live = b.finished[i] ? 0 : 1;
    b.meta.tok_seq[i] = i;
    b.meta.tok_pos[i] = pos;
    b.meta.tok_live[i] = live;
    b.meta.sample_row[i] = i;
    b.meta.sample_pos[i] = pos + 1;
    b.meta.sample_on[i] = live;
    return;
  }
  const int n_shares = b.n_shares, max_blocks = b.max_blocks;
  const bool team = b.team;
  const int32_t *shared = b.shared, *block_table = b.block_table;
  int32_t *unit_prefix = b.unit_prefix, *hdr = b.plan_hdr;
  __shared__ int sh[1024];
  __shared__ int carry, n_live;
  const int tid = threadIdx.x;
  const SharedView sv = shared_view(shared, n_seqs, Hkv);
  if (tid == 0) carry = n_live = 0;
  __syncthreads();
  for (int base = 0; base < n_seqs; base += 1024) {
    const int i = base + tid;
    // units of the sequence's own pairs: those after the ones that prefix tiles serve
    const int v = (i < n_seqs && !b.finished[i]) ? (ctx[i] + 1 + 31) / 32 - shared_units_of(sv, i, ctx[i]) : 0;
    sh[tid] = v;
    const int live_here = __popcll(__ballot(v > 0));
    if ((tid & 63) == 0 && live_here) atomicAdd(&n_live, live_here);
    __syncthreads();
    const int count = min(1024, n_seqs - base);
    for (int o = 1; o < count; o <<= 1) {
      const int t = tid >= o ? sh[tid - o] : 0;
      __syncthreads();
      sh[tid] += t;
      __syncthreads();
    }
    if (i < n_seqs) unit_prefix[i] = carry + sh[tid] - v;
    __syncthreads();
    if (tid == 0) carry += sh[count - 1];
    __syncthreads();
  }
  const int per_head = carry;
  if (tid == 0) unit_prefix[n_seqs] = per_head;
  __syncthreads();                                   // the prefix is read back below, from LDS if it is all there
  auto prefix = [&](int i) { return n_seqs > 1024 ? unit_prefix[i] : i ? sh[i - 1] : 0; };
  const int total = per_head * Hkv;
  // Share sizes differ by at most one unit: the units of the step are dealt out evenly and the first H shares take the
  // remainder, one unit each.  A share per wave is never empty, and there are on average at most MERGE_AT_ONCE of them per
  // live pair, the parts that the merge takes in one round trip: a lone sequence would leave it a part per unit otherwise
  // (4B shape, one sequence of 3000 keys, attention + merge: 2 units per share 15.0 us, 3 14.7, 6 17.3; the limit makes
  // it 3).  A pair far longer than the others has more parts than the average.
  const int n = team ? n_shares : max(1, min(min(n_shares, total), MERGE_AT_ONCE * n_live * Hkv));
  const int q = total / n, H = total % n;
  const int CA = q + 1, CB = q;
  if (tid == 0) { hdr[0] = CA; hdr[1] = total; hdr[2] = CB; hdr[3] = H; }
  const Shares shr = Shares{CA, CB, H, total};
  for (int w = tid; w < n_shares; w += 1024) {
    const int u0 = shr.start(w);
    int lo = 0, hi = n_seqs - 1;                     // largest s with Hkv * prefix[s] <= u0
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (Hkv * prefix(mid) <= u0) lo = mid; else hi = mid - 1;
    }
    int32_t* r = b.share_start + (size_t)w * SHARE_WORDS;
    const int end = min(total, shr.start(w + 1));
    if (u0 >= end) { r[6] = r[7] = 0; continue; }
    const int base = Hkv * prefix(lo), np = prefix(lo + 1) - prefix(lo), c = ctx[lo];
    const int kvh = (u0 - base) / np, pb = u0 - base - kvh * np, first = shared_units_of(sv, lo, c);
    const int last = min(np, end - (u0 - pb)) - 1;   // last unit of the first segment
    int32_t blocks[2 * SHARE_FIRST_UNITS];
#pragma unroll
    for (int i = 0; i < 2 * SHARE_FIRST_UNITS; ++i) {
      const int j = 2 * (first + min(pb + i / 2, last)) + (i & 1);
      const int32_t id = block_table[(size_t)lo * max_blocks + min(j, max_blocks - 1)];
      blocks[i] = j < max_blocks ? id : -1;
    }
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    static_assert(SHARE_WORDS == 16, "four stores");
    i32x4* out = reinterpret_cast<i32x4*>(r);
    out[0] = i32x4{lo, kvh, c, first};
    out[1] = i32x4{np, pb, u0, end};
    out[2] = i32x4{blocks[0], blocks[1], blocks[2], blocks[3]};
    out[3] = i32x4{blocks[4], blocks[5], blocks[6], blocks[7]};
  }
}

}  // namespace

hipError_t decode_begin(DecodeBeginArgs b, int n_wgs, hipStream_t st) {
  const int waves = 4 * n_wgs < ATTN_SHARES_MAX ? 4 * n_wgs : ATTN_SHARES_MAX;   // a larger grid leaves waves idle
  b.n_shares = b.team ? n_wgs : waves;
  hipLaunchKernelGGL(decode_begin_kernel, dim3(1 + b.n_seqs), dim3(1024), 0, st, b);
  return hipGetLastError();
}

template <int HD, int PL, int FMT, int NCT>
static void launch_prefix_columns(const AttnDecodeArgs& a, dim3 grid, hipStream_t st) {
  static std::once_flag raised;                      // above the default limit of 64 KB per workgroup
  constexpr int lds = PrefixLds<HD, NCT, PL>::BYTES;
  std::call_once(raised, [] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_decode_prefix_kernel<HD, PL, FMT, NCT>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  });
  hipLaunchKernelGGL((attn_decode_prefix_kernel<HD, PL, FMT, NCT>), grid, dim3(256), lds, st, a);
}
template <int HD, int PL, int FMT>
static void launch_prefix(const AttnDecodeArgs& a, dim3 grid, hipStream_t st) {
  // one column tile holds all members when there is one query head per KV head; two otherwise
  if (shared_prefix_members(a.Hq / a.Hkv) * (a.Hq / a.Hkv) <= 16) launch_prefix_columns<HD, PL, FMT, 1>(a, grid, st);
  else launch_prefix_columns<HD, PL, FMT, 2>(a, grid, st);
}

hipError_t attention_decode_prefix(const AttnDecodeArgs& a, hipStream_t st) {
  if (!a.shared) return hipSuccess;
  dim3 grid(a.n_prefix_wgs);
  const bool two = a.q.planes == 2;
  if (a.o.dtype == DT_F16) {
    if (a.hd == 128) launch_prefix<128, 1, DT_F16>(a, grid, st);
    else launch_prefix<64, 1, DT_F16>(a, grid, st);
  } else if (a.hd == 128) {
    if (two) launch_prefix<128, 2, DT_BF16>(a, grid, st);
    else launch_prefix<128, 1, DT_BF16>(a, grid, st);
  } else {
    if (two) launch_prefix<64, 2, DT_BF16>(a, grid, st);
    else launch_prefix<64, 1, DT_BF16>(a, grid, st);
  }
  return hipGetLastError();
}

template <int HD, int PL, int FMT>
static void launch_decode(const AttnDecodeArgs& a, hipStream_t st) {
  if (a.team) hipLaunchKernelGGL((attn_decode_team_kernel<HD, PL, FMT>), dim3(a.n_wgs), dim3(256), 0, st, a);
  else hipLaunchKernelGGL((attn_decode_kernel<HD, PL, FMT>), dim3(a.n_wgs), dim3(256), 0, st, a);
}

hipError_t attention_decode(const AttnDecodeArgs& a, hipStream_t st) {
  const bool two = a.q.planes == 2;
  // formats built: bf16 with one or two terms, fp16 with one term (checked when the model is created)
  if (a.o.dtype == DT_F16) {
    if (a.hd == 128) launch_decode<128, 1, DT_F16>(a, st);
    else launch_decode<64, 1, DT_F16>(a, st);
  } else if (a.hd == 128) {
    if (two) launch_decode<128, 2, DT_BF16>(a, st);
    else launch_decode<128, 1, DT_BF16>(a, st);
  } else {
    if (two) launch_decode<64, 2, DT_BF16>(a, st);
    else launch_decode<64, 1, DT_BF16>(a, st);
  }
  return hipGetLastError();
}

template <int HD>
static void launch_merge(const AttnDecodeArgs& a, hipStream_t st) {
  const dim3 grid(a.n_seqs * a.Hkv);
  const int slices = (a.Hq / a.Hkv) * HD / 8;        // 8-feature slices of a pair's heads: at most 16 * 128 / 8 = 256
  const int threads = (slices + 63) / 64 * 64;
  auto lds = [&](int groups) { return (size_t)(groups - 1) * slices * 10 * sizeof(float); };
  if (a.team) hipLaunchKernelGGL((attn_decode_merge_kernel<HD, 1>), grid, dim3(threads), lds(1), st, a);
  else if ((int)grid.x >= MERGE_MANY) hipLaunchKernelGGL((attn_decode_merge_kernel<HD, 2>), grid, dim3(threads * 2), lds(2), st, a);
  else hipLaunchKernelGGL((attn_decode_merge_kernel<HD, MERGE_GROUPS_MAX>), grid, dim3(threads * MERGE_GROUPS_MAX),
                          lds(MERGE_GROUPS_MAX), st, a);
}

hipError_t attention_decode_merge(const AttnDecodeArgs& a, hipStream_t st) {
  if (a.hd == 128) launch_merge<128>(a, st);
  else launch_merge<64>(a, st);
  return hipGetLastError();
}

}  // namespace rlx
