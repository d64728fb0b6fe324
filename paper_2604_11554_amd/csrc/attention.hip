// Prefill attention over the paged 16-bit KV pool.  A workgroup of four waves takes ATTN_QTILE = 64 consecutive query
// positions of one sequence for NCT heads of one KV group: wave w owns the 16 positions q0 + 16 w of the heads (a column
// tile per head, causal mask per column) and walks all keys itself, so there is no merge; the pages (32 keys per step)
// pass through LDS once for all waves, NB steps deep, one barrier per step.
// What bounds it: LDS reads, matrix products and softmax arithmetic take about the same time each, and the waves of a
// workgroup do them in step.  Two small workgroups per compute unit, each with its own barrier, drift apart and overlap
// them; one workgroup of eight waves and four heads did not (measured per layer: 30B-A3B shape, 16 x 128 tokens after 4900
// cached ones 544 us, with two workgroups 511; 4B shape, 32 565 tokens 884 -> 720; both 765 and 1145 at the start).
// Products of the next step's scores interleaved with this step's softmax in program order were slower (702 us).
// The hardware copies the pages into LDS (no registers, and no wait between a page's block-table entry and its load:
// the entries of the next 64 pages sit in a register, picked by lane number, the 64 after them in a second one).  The
// copies permute 16-byte chunks so that no fragment read meets a bank twice: K rows by the row number, V^T rows (32
// bytes) as the first chunks of sixteen rows and then their second ones.  (V^T as it lies in the page cost 60 % of the
// LDS cycles: SQ_LDS_BANK_CONFLICT / SQ_LDS_IDX_ACTIVE; 611 -> 544 us on the first of the calls above.)
#include "attn_core.h"
#include "lds_copy.h"

#include <mutex>

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

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15, g = lane >> 4;
  const int group = a.Hq / a.Hkv;

  if ((int)blockIdx.x >= a.n_qtiles[0]) return;      // uniform over the workgroup
  const int seq = a.qtile_seq[blockIdx.x];
  const int q0 = a.qtile_q0[blockIdx.x] + 16 * wave;  // this wave's first query position
  const int passes = (group + NCT - 1) / NCT;
  const int kvh = blockIdx.y / passes;
  const int hbase = (blockIdx.y % passes) * NCT;
  const int ctx = a.ctx_lens[seq];
  const int nq = a.cu_seqlens[seq + 1] - a.cu_seqlens[seq];
  const bool tile_live = q0 < nq && hbase < group;
  const int key_end = ctx + min(q0 + 16, nq);                                  // keys this wave's columns can see
  const int key_end_wg = ctx + min(a.qtile_q0[blockIdx.x] + ATTN_QTILE, nq);   // ... and the workgroup's last wave
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
  int voff[P];                                       // element offset of the lane's chunk inside its page
#pragma unroll
  for (int i = 0; i < P; ++i) {
    const int f = (wave + NW * i) % (COPIES / 2);    // KB of the page
    const int chunk = f * 64 + lane;                 // LDS slot, in 16-byte units
    const int row = chunk / RCH, slot = chunk % RCH;
    // K: row's chunks permuted; V^T, 16 features at a time: the first chunks (tokens 0..7) of their rows, then the second
    const int v = chunk - 16 * RCH;
    voff[i] = (row < 16 ? row * RCH + (slot ^ (RCH == 16 ? row : (row >> 1) & 7))
                        : 16 * RCH + ((v >> 5) * 16 + (v & 15)) * 2 + ((v >> 4) & 1)) * 8;
  }
  uint32_t ok_bits = 0;                              // validity of the two pages of the steps in LDS, two bits per step
  auto issue = [&](int pi, int buf) {                // past the end: the first page of the pool, marked invalid
    if (2 * pi - win >= 64) { tw0 = tw1; win += 64; tw1 = load_window(win + 64); }
    const int rel = 2 * pi - win;
    int64_t b0 = pi < n_pairs ? __builtin_amdgcn_readlane(tw0, rel & 63) : -1;
    int64_t b1 = pi < n_pairs ? __builtin_amdgcn_readlane(tw0, (rel + 1) & 63) : -1;
    const bool ok0 = b0 >= 0 && b0 < a.n_blocks, ok1 = b1 >= 0 && b1 < a.n_blocks;
    if (!ok0) b0 = 0;                                // keep the copies in bounds; scores are masked
    if (!ok1) b1 = b0;
    ok_bits = (ok_bits >> 2) | (((ok0 ? 1u : 0u) | (ok1 ? 2u : 0u)) << (2 * (NB - 1)));
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const int f = wave + NW * i;
      const int64_t b = f < COPIES / 2 ? b0 : b1;
      copy_to_lds(a.pool_layer + ((size_t)b * a.Hkv + kvh) * PAGE + voff[i], lds0 + buf * STAGE * 2 + f * 1024);
    }
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
  for (; pi < n_my; ++pi) {                          // n_my <= n_pairs
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
      vf[dt] = load_2x4(kv + off, kv + PAGE + off);
    }
    const bool ok0 = ok_bits & 1u, ok1 = ok_bits & 2u;
    pair_step<HD, NCT, PL, FMT>(st, k0, k1, vf, q_term, 32 * pi, 32 * pi + 16, ok0, ok1, key_end, pos_col,
                                ok0 && ok1 && 32 * pi + 31 <= ctx + q0, scale, g);
    buf = buf + 1 == NB ? 0 : buf + 1;
  }
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
  hipLaunchKernelGGL((attn_prefill_kernel<HD, NCT, PL, FMT>), dim3(a.max_qtiles, a.Hkv * passes), dim3(256),
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
