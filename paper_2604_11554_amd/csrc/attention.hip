// Prefill attention over the paged 16-bit KV pool.  A workgroup of four waves takes ATTN_QTILE = 64 consecutive query
// positions of one sequence for NCT heads of one KV group: wave w owns the 16 positions q0 + 16 w of the heads (a column
// tile per head, causal mask per column) and walks all keys itself, so there is no merge; the pages (32 keys per step)
// pass through LDS once for all waves, NB steps deep, one barrier per step.
// What bounds it: instruction issue.  With two waves per SIMD an instruction of any kind takes its wave's turn, so a step costs
// its ~480 instructions (64 products, 286 vector, 140 scalar in the worst step; LDS reads and products alone are half of that),
// and the waves of a workgroup do them in step.  Two small workgroups per compute unit, each with its own barrier, drift apart and
// overlap; one workgroup of eight waves and four heads did not.  us per layer, at the start / with two workgroups / with fewer
// instructions (no canonicalised maxima, no moves of V^T, short address arithmetic) / with units balanced: 30B-A3B shape, 16 x 128
// tokens after 2900 to 6900 cached ones 765 / 511 / 448 / 357; 4B shape, 32 565 tokens 1145 / 720 / 637 / 562.
// Products of the next step's scores interleaved with this step's softmax in program order were slower (702 us).
// The hardware copies the pages into LDS (no registers, and no wait between a page's block-table entry and its load:
// the entries of the next 64 pages sit in a register, picked by lane number, the 64 after them in a second one).  The
// copies permute 16-byte chunks so that no fragment read meets a bank twice: K rows by the row number, V^T rows (32
// bytes) as the first chunks of sixteen rows and then their second ones.  (V^T as it lies in the page cost 60 % of the
// LDS cycles: SQ_LDS_BANK_CONFLICT / SQ_LDS_IDX_ACTIVE; 611 -> 544 us on the first of the calls above.)
#include "attn_core.h"
#include "lds_copy.h"

#include <mutex>
#include <type_traits>

namespace rlx {
namespace {

constexpr int PREFILL_NB = 3;                          // steps in LDS: one being read, two on their way

template <int HD, int NCT, int PL, int FMT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_prefill_kernel(AttnArgs a) {
  constexpr int DT = HD / 16, KS = HD / 32, NW = 4, NB = PREFILL_NB;
  constexpr int PAGE = 2 * 16 * HD, KPART = 16 * HD, STAGE = 2 * PAGE;   // elements of a page, of its K rows, of a step
  constexpr int COPIES = STAGE * 2 / 1024, P = COPIES / NW;              // 1 KB copies per step, and per wave
  constexpr int RCH = HD / 8;                          // 16-byte chunks per K row
  static_assert(COPIES % NW == 0, "the waves share a step's copies evenly");
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const h16_t* lds_kv = reinterpret_cast<const h16_t*>(lds_raw);   // [NB][STAGE]
  // 8 bytes of V^T.  (Volatile: left to itself the compiler reads two features' of one page at once and then sorts the pairs
  // with a move per register, 24 a step.)
  auto read_v = [](const h16_t* p) { return *(const volatile __attribute__((address_space(3))) u32x2*)p; };

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15, g = lane >> 4;
  const int group = a.Hq / a.Hkv;

  // The grid runs over (tile, pass, KV head), the longest tiles first.  Where all workgroups are resident at once, two per
  // unit, the second of a unit takes its tile from the list's end, so that units get a long one and a short one
  // (30B-A3B shape, 16 x 128 tokens after 2900 to 6900 cached ones: 511 us a layer before, 368 with the list and the pairing).
  const int passes = (group + NCT - 1) / NCT, per_tile = passes * a.Hkv;
  const int live = a.n_qtiles[0] * per_tile;
  int id = blockIdx.x;
  if (id >= live) return;                            // uniform over the workgroup
  if (id >= a.n_units && live <= 2 * a.n_units) id = live - 1 - (id - a.n_units);
  const int tile = id / per_tile, kvh = id % per_tile % a.Hkv, hbase = id % per_tile / a.Hkv * NCT;
  const int seq = a.qtile_seq[tile], tile_q0 = a.qtile_q0[tile];
  const int q0 = tile_q0 + 16 * wave;                // this wave's first query position
  const int ctx = a.ctx_lens[seq];
  const int nq = a.cu_seqlens[seq + 1] - a.cu_seqlens[seq];
  const bool tile_live = q0 < nq && hbase < group;
  const int key_end = ctx + min(q0 + 16, nq);                                  // keys this wave's columns can see
  const int key_end_wg = ctx + min(tile_q0 + ATTN_QTILE, nq);   // ... and the workgroup's last wave
  const int blk_end = (key_end_wg + 15) >> 4;        // exclusive
  const int n_pairs = (blk_end + 1) >> 1;

  // ---- block table: lane i of tw0 holds entry win + i, of tw1 entry win + 64 + i; entries that do not exist are -1 ----
  const int32_t* table = a.block_table + (size_t)seq * a.max_blocks;
  const int t_end = min(blk_end, a.max_blocks);
  auto load_window = [&](int first) {
    const int j = first + lane;
    const int32_t v = table[min(j, a.max_blocks - 1)];
    return j < t_end ? v : -1;
  };
  int win = 0;
  int32_t tw0 = load_window(0), tw1 = load_window(64);

  // ---- query fragments and per-column limits ----
  h16x8 qf[PL][NCT][KS];
  int pos_col[NCT];
  bool col_ok[NCT];
  int trow[NCT], head[NCT];
#pragma unroll
  for (int c = 0; c < NCT; ++c) {
    head[c] = kvh * group + hbase + c;
    col_ok[c] = (hbase + c < group) && (q0 + c16 < nq);
    trow[c] = a.cu_seqlens[seq] + q0 + c16;
    pos_col[c] = ctx + q0 + c16;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const h16_t* src = a.q.p + ((size_t)trow[c] * a.Hq + head[c]) * HD + 32 * ks + 8 * g;
#pragma unroll
      for (int p = 0; p < PL; ++p) qf[p][c][ks] = col_ok[c] ? load_h16x8(src + p * a.q.plane) : zero_h16x8();
    }
  }
  auto q_term = [&](int p, int c, int ks) -> h16x8 { return qf[p][c][ks]; };

  WaveState<HD, NCT> st;
  st.reset();
  const float scale = rsqrtf((float)HD);

  // ---- copies: wave w takes KBs w, w + NW, ... of a step's two pages ----
  const uint32_t lds0 = lds_address(lds_raw);
  static_assert(P % 2 == 0, "the first half of a wave's copies is of the first page");
  uint32_t voff[P / 2];                              // byte offset of the lane's chunk inside its page
#pragma unroll
  for (int i = 0; i < P / 2; ++i) {
    const int chunk = (wave + NW * i) * 64 + lane;   // LDS slot, in 16-byte units
    const int row = chunk / RCH, slot = chunk % RCH;
    // K: row's chunks permuted; V^T, 16 features at a time: the first chunks (tokens 0..7) of their rows, then the second
    const int v = chunk - 16 * RCH;
    voff[i] = (row < 16 ? row * RCH + (slot ^ (RCH == 16 ? row : (row >> 1) & 7))
                        : 16 * RCH + ((v >> 5) * 16 + (v & 15)) * 2 + ((v >> 4) & 1)) * 16;
  }
  uint32_t ok_bits = 0;                              // validity of the two pages of the steps in LDS, two bits per step
  const uint32_t n_blocks = (uint32_t)min(a.n_blocks, (int64_t)0x7FFFFFFF);
  const uint32_t lds_w = lds0 + wave * 1024;
  // Scalar work is kept short: with two waves per SIMD an instruction of any kind takes its wave's turn.  Entries past the
  // sequence's end are -1 in the windows; such a step copies the first page of the pool and is marked invalid.
  auto issue = [&](int pi, int buf) {
    if (2 * pi - win >= 64) { tw0 = tw1; win += 64; tw1 = load_window(win + 64); }
    const int rel = 2 * pi - win;
    uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane(tw0, rel & 63), b1 = (uint32_t)__builtin_amdgcn_readlane(tw0, (rel + 1) & 63);
    const bool ok0 = b0 < n_blocks, ok1 = b1 < n_blocks;
    if (!ok0) b0 = 0;                                // keep the copies in bounds; scores are masked
    if (!ok1) b1 = b0;
    ok_bits = (ok_bits >> 2) | (((ok0 ? 1u : 0u) | (ok1 ? 2u : 0u)) << (2 * (NB - 1)));
    const uint32_t hkv = (uint32_t)a.Hkv;            // a pool of more than 2^32 pages of a head does not exist
    const h16_t* p0 = a.pool_layer + (size_t)(b0 * hkv + (uint32_t)kvh) * PAGE;
    const h16_t* p1 = a.pool_layer + (size_t)(b1 * hkv + (uint32_t)kvh) * PAGE;
    const uint32_t dst = lds_w + (uint32_t)buf * (STAGE * 2);
#pragma unroll
    for (int i = 0; i < P; ++i) copy_to_lds(i < P / 2 ? p0 : p1, voff[i % (P / 2)], dst + NW * i * 1024);
  };

#pragma unroll
  for (int s = 0; s < NB - 1; ++s) issue(s, s);
  const int n_my = tile_live ? (key_end + 31) >> 5 : 0;   // steps up to the wave's last column; uniform
  int pi = 0, buf = 0, fbuf = NB - 1;
  auto next_step = [&]() {                           // step pi's pages are in LDS, the last step's are read
    wait_copies_and_barrier<(NB - 2) * P>();
    issue(pi + NB - 1, fbuf);
    fbuf = fbuf + 1 == NB ? 0 : fbuf + 1;
    __builtin_amdgcn_sched_barrier(0);
  };
  auto step = [&](auto late) {
    next_step();
    const h16_t* kv = lds_kv + buf * STAGE;
    h16x8 k0[KS], k1[KS], vf[DT];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int off = c16 * HD + ((4 * ks + g) ^ (RCH == 16 ? c16 : (c16 >> 1) & 7)) * 8;
      k0[ks] = load_h16x8(kv + off);
      k1[ks] = load_h16x8(kv + PAGE + off);
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const int off = KPART + dt * 256 + (g >> 1) * 128 + c16 * 8 + (g & 1) * 4;
      const u32x2 v0 = read_v(kv + off), v1 = read_v(kv + PAGE + off);
      vf[dt] = h16x8{v0[0], v0[1], v1[0], v1[1]};
    }
    const bool ok0 = ok_bits & 1u, ok1 = ok_bits & 2u;
    pair_step<HD, NCT, PL, FMT, decltype(late)::value>(st, k0, k1, vf, q_term, 32 * pi, 32 * pi + 16, ok0, ok1, key_end, pos_col,
                                                       ok0 && ok1 && 32 * pi + 31 <= ctx + q0, scale, g);
    buf = buf + 1 == NB ? 0 : buf + 1;
  };
  for (const int early = min(n_my, 32); pi < early; ++pi) step(std::false_type());   // n_my <= n_pairs
  for (; pi < n_my; ++pi) step(std::true_type());
  for (; pi < n_pairs; ++pi) next_step();            // waves of smaller positions keep copying for the others
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no copy may outlive the workgroup's LDS
  if (!tile_live) return;
  st.finish_denominators();
#pragma unroll
  for (int c = 0; c < NCT; ++c) store_column<HD, NCT, PL, FMT>(st, c, a.o, trow[c], head[c], g, col_ok[c]);
}

}  // namespace

template <int HD, int PL, int FMT>
static void launch_prefill(const AttnArgs& a, hipStream_t st) {
  constexpr int NCT = 2;
  constexpr size_t lds = (size_t)PREFILL_NB * 2 * 2 * 16 * HD * sizeof(h16_t);   // steps of two pages
  static std::once_flag raised;                      // above the default limit of 64 KB per workgroup
  std::call_once(raised, [] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_prefill_kernel<HD, NCT, PL, FMT>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  });
  const int group = a.Hq / a.Hkv;
  const int passes = (group + NCT - 1) / NCT;
  hipLaunchKernelGGL((attn_prefill_kernel<HD, NCT, PL, FMT>), dim3(a.max_qtiles * a.Hkv * passes), dim3(256),
                     lds, st, a);
}

hipError_t attention_prefill(const AttnArgs& a, hipStream_t st) {
  const bool two = a.q.planes == 2;
  // formats built: bf16 with one or two terms, fp16 with one term (checked when the model is created)
  if (a.o.dtype == DT_F16) {
    if (a.hd == 128) launch_prefill<128, 1, DT_F16>(a, st);
    else launch_prefill<64, 1, DT_F16>(a, st);
  } else if (a.hd == 128) {
    if (two) launch_prefill<128, 2, DT_BF16>(a, st);
    else launch_prefill<128, 1, DT_BF16>(a, st);
  } else {
    if (two) launch_prefill<64, 2, DT_BF16>(a, st);
    else launch_prefill<64, 1, DT_BF16>(a, st);
  }
  return hipGetLastError();
}

}  // namespace rlx
