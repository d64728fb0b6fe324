// C ABI of the rollout library: handle lifetime, argument validation, workspace
// carving and the launch sequence of one prefill chunk / decode step.
#include "../../include/relax_rollout.h"

#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <mutex>
#include <new>
#include <vector>

#include "kernels.h"

using namespace rlx;

namespace {

thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

#define RLX_HIP(expr)                                                                        \
  do {                                                                                       \
    hipError_t e_ = (expr);                                                                  \
    if (e_ != hipSuccess) return fail(RLX_EHIP, "%s: %s", #expr, hipGetErrorString(e_));     \
  } while (0)

// Optional timing aid: launches of one kernel class are bracketed with caller-owned events.
struct ProfState {
  int cls = 0;
  void* const* start = nullptr;
  void* const* stop = nullptr;
  int n = 0, used = 0, stride = 1, seen = 0;
};
ProfState g_prof;

#define RLX_LAUNCH(cls_, expr)                                                               \
  do {                                                                                       \
    bool p_ = false;                                                                         \
    if (g_prof.cls == (cls_) && g_prof.used < g_prof.n) p_ = (g_prof.seen++ % g_prof.stride) == 0; \
    if (p_) RLX_HIP(hipEventRecord((hipEvent_t)g_prof.start[g_prof.used], st));              \
    RLX_HIP(expr);                                                                           \
    if (p_) RLX_HIP(hipEventRecord((hipEvent_t)g_prof.stop[g_prof.used++], st));             \
  } while (0)

size_t align_up(size_t v, size_t a = 256) { return (v + a - 1) / a * a; }

// Fixed scratch for callers that cannot allocate (rollout_decode_step_static): one array per GPU, resident from
// the moment the library's code is loaded on that GPU until the process ends.  Host code never uses the array's
// name as an address: scratch_on_device() asks the runtime once per device, with that device current, where that
// device's copy lives, and every launch receives the pointer it returned.
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[RLX_STATIC_WORKSPACE_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[MAX_DEVICES] = {};

// device `dev` must be the current device
hipError_t scratch_on_device(int dev, void** out) {
  *out = nullptr;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

struct rlx_model {
  rlx_model_config cfg;
  const h16_t *embed, *lm_head, *final_norm;
  std::vector<const h16_t*> attn_norm, wq, wk, wv, wo, q_norm, k_norm, ffn_norm, w_gate_up, w_down, w_router;
  double* inv_freq;   // device, [head_dim / 2]
  int device;
  int n_units;        // compute units of the device
  int attn_wgs;       // decode attention grid: two workgroups per compute unit
  uint64_t weight_version;   // tag of the installed weights (rlx_model_set_weights)
  void* static_ws;           // this device's fixed scratch array (rollout_decode_step_static)
};

namespace {

int prefix_wgs(const rlx_model* m) { return 2 * m->n_units; }   // workgroups of the prefix tiles: all resident

struct Workspace {
  TokenMeta meta;
  float* h;          // [T, d]
  h16_t* xb;        // [planes][T, d]; every 16-bit activation buffer below has `planes` copies
  float* router;     // [planes][T, E] router logits (MoE)
  float* qkv;        // [planes][T, qkv_dim]
  h16_t* q;         // [T, q_dim]
  h16_t* ob;        // [T, q_dim]
  float* attn_part;  // [ATTN_SHARES_MAX][2][Hq/Hkv][hd+4] decode partials of straddling (sequence, KV head) pairs
  int32_t *attn_prefix, *attn_share_start, *attn_hdr;   // decode attention plan
  float* attn_seq_part;   // [S][Hkv][Hq/Hkv][hd+4] own part of a pair that prefix tiles precede
  float* attn_pre_part;   // [shared_prefix_max_tiles][SP_COLS][hd+4] parts of the shared-prefix tiles
  float* planes;     // split-K planes of the o / down projections
  h16_t* act;       // dense [T, F]; MoE [T*top_k, Fe]
  float* moe_y;      // [T*top_k, d]
  int32_t* topk_idx; float* topk_w;
  int32_t *group_ws, *group_off, *sorted_token, *pair_pos;
  float* x_ss;                        // [T][4] sums of squares of the row quarters (norm of short calls, Act::ss)
  GroupItems items;                   // (expert, row tile) list of the grouped GEMMs of long calls
  h16_t* x_lm;      // [S, d]
  float* lm_part;    // [S][tiles][4]
  size_t bytes;
};

// rows per LM-head pass of rollout_score_chunk: passes of a thousand rows leave a twentieth of the device idle at their end,
// passes of 256 a quarter (30B-A3B shape, 151 936 x 2048: 256 rows 300 us, 1024 rows 1007); short calls stay with 256
constexpr int SCORE_ROWS = 1024;
int score_rows_max(int T) { return T <= 256 ? 256 : (T < SCORE_ROWS ? T : SCORE_ROWS); }
constexpr int ATTN_WGS_MAX = 1024;   // decode attention grid limit

// Calls of more than 128 tokens (MoE: 256) on two-term bf16 activations carry them in rows and take the long-call GEMMs.
bool two_term(const rlx_model_config& c) { return c.activation_split && c.dtype == RLX_DTYPE_BF16; }
int short_tokens(const rlx_model_config& c) { return two_term(c) && !c.n_experts ? 128 : 256; }   // of the calls that split K in up to 16
bool long_call(const rlx_model_config& c, int T) { return T > short_tokens(c) && two_term(c); }
// ... and so do LM heads of more than 64 rows (151 936 x 2560, one draw per row: 96 rows 234 -> 209 us, 256 rows 509 -> 435;
// 64 rows 153 in the short form, 161 at best in long ones)
bool rows_lmhead(const rlx_model_config& c, int rows) { return rows > 64 && two_term(c); }
// Decode attention of MoE policies keeps a share of the keys per workgroup: in a share per wave the sums come in another
// order, and the last bits of the router's input decide near-ties of the routing (30B-A3B shape, 128 sequences of 1530
// keys: one token took its ninth expert for its eighth, which moved the batch's logits by 3 % of their norm).
bool attn_by_team(const rlx_model_config& c) { return c.n_experts > 0; }
Act call_act(const rlx_model_config& c, h16_t* p, int T, int K, bool rows) {
  return rows ? make_act_rows(p, T, K) : make_act(p, T, K, c.activation_split ? 2 : 1, c.dtype);
}

// Split-K planes per token of an output of up to d_model features (the o and down projections) and of the wider q|k|v in
// long calls: as many as keep the planes under 16384 (8192) rows, at most eight (four), and two (one) however long the
// call.  Long calls of MoE policies keep their sums whole: the other order of sums would change the last bits of the
// router's input, which decide near-ties of the routing, and 128 x 128 tiles fill the device there without planes (30B-A3B
// shape, 2048 tokens: output projection 64 us whole, 63 in two planes).  `lean`: two (one) at any length, for calls that
// would not fit their scratch otherwise.
int long_planes(const rlx_model_config& c, int T, bool wide, bool lean) {
  if (c.n_experts) return 1;
  const int most = wide ? 4 : 8, n = (wide ? 8192 : 16384) / T, least = wide ? 1 : 2;
  return lean || n < least ? least : (n > most ? most : n);
}
// rows of the planes of a call of T tokens: sixteen per token in short calls, one in longer ones that carry one term
size_t plane_rows(const rlx_model_config& c, int T, bool wide, bool lean) {
  if (T <= short_tokens(c)) return (size_t)gemm_max_splits() * T;
  return (size_t)(two_term(c) ? long_planes(c, T, wide, lean) : 1) * T;
}
// ... and at most of a call of up to T tokens
size_t plane_rows_up_to(const rlx_model_config& c, int T, bool wide) {
  const size_t shrt = (size_t)gemm_max_splits() * (T < short_tokens(c) ? T : short_tokens(c));
  size_t lng = (size_t)T;
  if (two_term(c) && !c.n_experts) {
    const size_t most = (wide ? 4 : 8) * lng, cap = wide ? 8192 : 16384, least = (wide ? 1 : 2) * lng;
    lng = least > cap ? least : (most < cap ? most : cap);
  }
  return shrt > lng ? shrt : lng;
}

// Carve the workspace; with base == nullptr only the size is computed.  S sequences; T: the larger of S and the number of
// tokens; `planes`: rows of the split-K planes, narrow and wide.
struct PlaneRows { size_t narrow, wide; };
PlaneRows call_planes(const rlx_model_config& c, int tokens, bool lean = false) {
  return {plane_rows(c, tokens, false, lean), plane_rows(c, tokens, true, lean)};
}
Workspace carve(const rlx_model_config& c, char* base, int S, int T, const PlaneRows& planes) {
  Workspace w = {};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? base + off : nullptr;
    off += align_up(bytes);
    return p;
  };
  const int qdim = c.n_q_heads * c.head_dim, kvdim = c.n_kv_heads * c.head_dim;
  const int qkv_dim = qdim + 2 * kvdim;
  const int QT = T / 16 + S + 1;
  w.meta.tok_seq = (int32_t*)take((size_t)T * 4);
  w.meta.tok_pos = (int32_t*)take((size_t)T * 4);
  w.meta.tok_live = (uint8_t*)take((size_t)T);
  w.meta.sample_row = (int32_t*)take((size_t)S * 4);
  w.meta.sample_pos = (int32_t*)take((size_t)S * 4);
  w.meta.sample_on = (uint8_t*)take((size_t)S);
  w.meta.qtile_seq = (int32_t*)take((size_t)QT * 4);
  w.meta.qtile_q0 = (int32_t*)take((size_t)QT * 4);
  w.meta.n_qtiles = (int32_t*)take(4);
  w.meta.tok_iota = (int32_t*)take((size_t)T * 4);
  w.meta.rope_cs = (float2*)take((size_t)T * (c.head_dim / 2) * sizeof(float2));
  w.h = (float*)take((size_t)T * c.d_model * 4);
  const int PL = c.activation_split ? 2 : 1;
  auto act_bytes = [&](int rows, int K, bool in_rows) {
    const size_t frag = frag_act_elems(rows, K, PL) * 2, r = in_rows ? act_rows_elems(rows, K) * 2 : 0;
    return frag > r ? frag : r;
  };
  const bool lng = long_call(c, T);
  w.xb = (h16_t*)take(act_bytes(T, c.d_model, lng));
  w.x_ss = (float*)take((size_t)T * NORM_PARTS * 4);
  w.router = c.n_experts ? (float*)take(planes.narrow * c.n_experts * 4) : nullptr;
  w.q = (h16_t*)take((size_t)PL * T * qdim * 2);
  w.ob = (h16_t*)take(act_bytes(T, qdim, lng));
  w.attn_prefix = (int32_t*)take((size_t)(S + 1) * 4);
  w.attn_hdr = (int32_t*)take(4 * 4);
  w.attn_seq_part = (float*)take((size_t)S * c.n_q_heads * (c.head_dim + 4) * 4);
  w.attn_pre_part = (float*)take((size_t)shared_prefix_max_tiles(S, c.n_kv_heads) * SP_COLS * (c.head_dim + 4) * 4);
  // Split-K planes of q|k|v and of the o and down projections.  Both are dead while decode attention runs (its queries
  // are rotated, the residual has taken the planes up), so its partials lie in the same memory.
  const size_t planes_at = off;
  w.qkv = (float*)take(planes.wide * qkv_dim * 4);
  w.planes = (float*)take(planes.narrow * c.d_model * 4);
  w.attn_part = w.qkv;
  const size_t attn_end = planes_at + align_up((size_t)ATTN_SHARES_MAX * 2 * (c.n_q_heads / c.n_kv_heads) * (c.head_dim + 4) * 4);
  if (off < attn_end) off = attn_end;
  if (c.n_experts) {
    const size_t P = (size_t)T * c.top_k;
    w.act = (h16_t*)take(act_bytes((int)P, c.d_ff_expert, lng));
    w.moe_y = (float*)take(P * c.d_model * 4);
    w.topk_idx = (int32_t*)take(P * 4);
    w.topk_w = (float*)take(P * 4);
    w.group_ws = (int32_t*)take(moe_group_workspace_words() * 4);
    w.group_off = (int32_t*)take((size_t)(c.n_experts + 1) * 4);
    w.sorted_token = (int32_t*)take(P * 4);
    w.pair_pos = (int32_t*)take(P * 4);
    w.items.tile_rows = gemm_long_item_rows((int)((P + c.n_experts - 1) / c.n_experts));
    w.items.max_items = (int)(P / w.items.tile_rows) + c.n_experts;   // at most one partial tile per expert
    const size_t item_room = (P / 64 + c.n_experts) * 4;              // of the smallest tile: does not fall as T grows
    w.items.expert = (int32_t*)take(item_room);
    w.items.tile = (int32_t*)take(item_room);
    w.items.count = (int32_t*)take(4);
  } else {
    w.act = (h16_t*)take(act_bytes(T, c.d_ff, lng));
  }
  // Behind the layers: rows and partials of the LM head.  A decode step has the records of its attention shares there, which its
  // first launch writes and its last layer reads, before the final norm writes the rows.
  const size_t lm_at = off;
  w.attn_share_start = base ? (int32_t*)(base + lm_at) : nullptr;
  const int score_rows = score_rows_max(T), lm_rows = S > score_rows ? S : score_rows;   // sampled rows, or a block of scored ones
  w.x_lm = (h16_t*)take(act_bytes(lm_rows, c.d_model, rows_lmhead(c, lm_rows)));
  // a part per 64 ids or more in the forms of many rows, per 32 in that of up to 64: there are at least 256 rows here
  w.lm_part = (float*)take((size_t)lm_rows * (two_term(c) ? (c.vocab + 63) / 64 : (c.vocab + 31) / 32) * 4 * 4);
  const size_t shares_end = lm_at + align_up((size_t)ATTN_SHARES_MAX * ATTN_SHARE_WORDS * 4);
  w.bytes = off > shares_end ? off : shares_end;
  return w;
}

size_t block_elems(const rlx_model_config& c) { return (size_t)c.n_kv_heads * 2 * 16 * c.head_dim; }

struct StepIO {
  int n_seqs, T;
  bool decode;
  const int32_t* tokens; const h16_t* input_embeds;
  const int32_t* cu_seqlens; const int32_t* ctx_lens;
  const int32_t* block_table; int max_blocks;
  const uint64_t* seeds; const float* temperature; const int32_t* max_ctx_len; const int32_t* forced;
  int32_t* out_tokens; float* out_logprobs; uint8_t* finished; int32_t* out_sampled;
  int32_t* out_routing; float* out_logits;
  int32_t* ctx_lens_rw;   // decode only
  // scoring (rollout_score_chunk): every chunk position is scored against score_targets, nothing is sampled
  bool score; const int32_t* score_targets; float* score_logprobs;
  const int32_t* replay_routing;   // optional [T, n_layers, top_k]
  const int32_t* shared_prefix;    // decode only, optional descriptor of shared prompt prefixes
  bool lean;                       // as few split-K planes as a long call can do with (long_planes)
};

int run_layers(const rlx_model* m, h16_t* pool, int64_t n_blocks, const Workspace& w, const StepIO& io,
               hipStream_t st) {
  const rlx_model_config& c = m->cfg;
  const int d = c.d_model, T = io.T;
  const int qdim = c.n_q_heads * c.head_dim, kvdim = c.n_kv_heads * c.head_dim, qkv_dim = qdim + 2 * kvdim;
  const int PL = c.activation_split ? 2 : 1;
  const int FMT = c.dtype;
  const bool lng = long_call(c, T), small = T <= 256 && !lng;
  Act xb = call_act(c, w.xb, T, d, lng);
  const Act ob = call_act(c, w.ob, T, qdim, lng);
  const RowAct qb = {w.q, (size_t)T * qdim, qdim, PL, FMT};

  if (!io.decode) RLX_HIP(embed_tokens(m->embed, c.vocab, d, io.tokens, io.input_embeds, T, w.h, FMT, st));

  // residual contribution produced by the previous sub-layer, folded into the next norm
  const float* pend_planes = nullptr; int pend_n = 0; bool pend_moe = false;
  // MoE decode batches: the gate/up GEMM reads the routing table itself and publishes the grouping (no grouping launch)
  const bool routed = c.n_experts && small && gemm_routed_form(c.n_experts, xb, T * c.top_k);
  // calls of up to 256 tokens: the norm runs as four workgroups per row (256 rows of 2560: 6.4 us; in one 8.9) and leaves
  // the row's common factor to the GEMMs that read xb (q|k|v, gate/up, router), which also keeps rows that two bf16 terms
  // hold exactly (embeddings) exact; not for fp16 (unnormalised rows would strain its range) and not where the grouped
  // gate/up goes through a row list
  if (T <= 256 && FMT == DT_BF16 && rmsnorm_in_parts(d) && (c.n_experts == 0 || routed)) { xb.ss = w.x_ss; xb.eps = c.rms_eps; }
  // y = x W^T into `y`: split-K planes that the next kernel adds.  q|k|v of long calls of up to 256 tokens (decode batches) comes
  // in all the planes it may have: keys and values are rounded to 16 bits right after, and with longer sums more of them
  // get the neighbouring code (K 2560, of six million values 1908 with the two planes that are fastest, 1573 with four, 1490
  // in calls of 64 tokens; logits of 256 rows, four layers: 2.5e-5 of their norm off a 64-bit computation with two, 2.3e-5 with
  // four and in the short form; eight layers, 129 rows: 1500 -> 1520 us a step, 256 rows 1910 both).
  const bool fine_qkv = T <= 256;
  // Form and planes of a product are the same in every layer: settled once per call (the search over 64 cuts of a short call's
  // product is 0.3 us of host time, six of them a layer).  Short-call form in dense policies only: MoE decode keeps its
  // sums in the order that its routing was recorded with.
  struct Plan { bool is_flow; FlowPlan flow; LongPlan lng; int planes; };
  auto plan_of = [&](int N, int K, bool wide) {
    Plan p = {small && c.n_experts == 0 && gemm_flow_store_form(N, K, T, m->n_units, PL, FMT), {}, {}, 1};
    if (p.is_flow) {
      p.flow = flow_store_plan(N, K, T, gemm_max_splits(), m->n_units, PL);
      p.planes = p.flow.splits;
    } else if (small) {
      p.planes = gemm_plan_splits(N, K, T, gemm_max_splits(), m->n_units, PL, FMT);
    } else if (lng) {
      p.lng = long_plan(N, K, T, long_planes(c, T, wide, io.lean), m->n_units, wide && fine_qkv);
      p.planes = p.lng.splits;
    }
    return p;
  };
  auto store = [&](const LinearW& lw, const Act& x, float* y, const Plan& p, const FlowNorm* nm = nullptr) {
    return p.is_flow ? gemm_flow_store(lw, x, T, y, lw.N, p.flow, st, nm)
           : lng     ? gemm_long_store(lw, x, T, y, lw.N, p.lng, st)
                     : gemm_store(lw, x, T, y, lw.N, p.planes, st);
  };
  const Plan p_qkv = plan_of(qkv_dim, d, true), p_o = plan_of(d, qdim, false);
  const Plan p_ffn = c.n_experts ? plan_of(c.n_experts, d, false) : plan_of(d, c.d_ff, false);   // router, or down
  float* h_at = w.h;                                  // where the residual stream is
  auto norm = [&](const h16_t* gain, const int32_t* rows, int n_rows, const Act& x, float* xf) -> hipError_t {
    NormArgs a = {};
    a.h = h_at; a.gain = gain; a.d = d; a.T = n_rows; a.T_total = T; a.eps = c.rms_eps; a.rows = rows;
    a.add = pend_planes; a.n_planes = pend_n;
    if (pend_moe) { a.moe_y = w.moe_y; a.pair_pos = w.pair_pos; a.topk_w = w.topk_w; a.top_k = c.top_k; }
    a.x = x; a.xf = xf;
    pend_planes = nullptr; pend_n = 0; pend_moe = false;
    return rmsnorm(a, st);
  };

  // Calls of few tokens: the products that read normalised rows make them themselves.  The residual stream then changes its place
  // with every addition, between w.h and the activation matrix that nothing else uses here (32 rows of 4 bytes per element, or of
  // two; at most sixteen rows of four are put there).
  const bool norm_inside = p_qkv.is_flow && flow_norm_form(T, d, p_o.planes, p_ffn.planes) &&
                           gemm_flow_swiglu_form(c.d_ff, T, m->n_units, PL, FMT);
  auto inner_norm = [&](const h16_t* gain) {
    FlowNorm f = {h_at, nullptr, pend_planes, pend_n, gain, c.rms_eps, nullptr};
    if (pend_planes) h_at = f.h_out = h_at == w.h ? (float*)w.xb : w.h;
    pend_planes = nullptr; pend_n = 0;
    return f;
  };

  for (int l = 0; l < c.n_layers; ++l) {
    FlowNorm nm = {};
    if (norm_inside) nm = inner_norm(m->attn_norm[l]);
    else RLX_LAUNCH(RLX_K_NORM, norm(m->attn_norm[l], nullptr, T, xb, nullptr));
    LinearW wqkv = {};
    wqkv.seg[0] = m->wq[l]; wqkv.rows[0] = qdim;
    wqkv.seg[1] = m->wk[l]; wqkv.rows[1] = kvdim;
    wqkv.seg[2] = m->wv[l]; wqkv.rows[2] = kvdim;
    wqkv.N = qkv_dim; wqkv.K = d;
    RLX_LAUNCH(RLX_K_QKV, store(wqkv, xb, w.qkv, p_qkv, norm_inside ? &nm : nullptr));

    h16_t* pool_layer = pool + (size_t)l * n_blocks * block_elems(c);
    RopeArgs r = {};
    r.qkv = w.qkv; r.n_planes = p_qkv.planes;
    r.q_gain = c.qk_norm ? m->q_norm[l] : nullptr; r.k_gain = c.qk_norm ? m->k_norm[l] : nullptr;
    r.rope_cs = w.meta.rope_cs;
    r.T = T; r.Hq = c.n_q_heads; r.Hkv = c.n_kv_heads; r.hd = c.head_dim;
    r.eps = c.rms_eps; r.tok_seq = w.meta.tok_seq; r.tok_pos = w.meta.tok_pos; r.tok_live = w.meta.tok_live;
    r.block_table = io.block_table; r.max_blocks = io.max_blocks;
    r.pool_layer = pool_layer; r.n_blocks = n_blocks; r.q_out = qb;
    RLX_LAUNCH(RLX_K_ROPE, qk_rope_append(r, st));
    if (io.decode) {
      AttnDecodeArgs at = {};
      at.q = qb; at.pool_layer = pool_layer; at.n_blocks = n_blocks;
      at.Hq = c.n_q_heads; at.Hkv = c.n_kv_heads; at.hd = c.head_dim;
      at.block_table = io.block_table; at.max_blocks = io.max_blocks; at.ctx_lens = io.ctx_lens;
      at.n_seqs = io.n_seqs; at.unit_prefix = w.attn_prefix; at.share_start = w.attn_share_start; at.plan_hdr = w.attn_hdr;
      at.team = attn_by_team(c); at.n_wgs = m->attn_wgs; at.part = w.attn_part; at.o = ob;
      at.shared = io.shared_prefix; at.seq_part = w.attn_seq_part; at.pre_part = w.attn_pre_part;
      at.n_prefix_wgs = prefix_wgs(m);
      RLX_LAUNCH(RLX_K_ATTN_PREFIX, attention_decode_prefix(at, st));
      RLX_LAUNCH(RLX_K_ATTN, attention_decode(at, st));
      RLX_LAUNCH(RLX_K_ATTN_MERGE, attention_decode_merge(at, st));
    } else {
      AttnArgs at = {};
      at.q = qb; at.pool_layer = pool_layer; at.n_blocks = n_blocks;
      at.Hq = c.n_q_heads; at.Hkv = c.n_kv_heads; at.hd = c.head_dim;
      at.block_table = io.block_table; at.max_blocks = io.max_blocks; at.ctx_lens = io.ctx_lens;
      at.cu_seqlens = io.cu_seqlens; at.qtile_seq = w.meta.qtile_seq; at.qtile_q0 = w.meta.qtile_q0;
      at.n_qtiles = w.meta.n_qtiles; at.max_qtiles = T / ATTN_QTILE + io.n_seqs + 1; at.n_units = m->n_units; at.o = ob;
      RLX_LAUNCH(RLX_K_ATTN, attention_prefill(at, st));
    }

    RLX_LAUNCH(RLX_K_OPROJ, store(linear1(m->wo[l], d, qdim), ob, w.planes, p_o));
    pend_planes = w.planes; pend_n = p_o.planes;

    if (norm_inside) nm = inner_norm(m->ffn_norm[l]);
    else RLX_LAUNCH(RLX_K_NORM, norm(m->ffn_norm[l], nullptr, T, xb, nullptr));
    if (c.n_experts == 0) {
      const Act act = call_act(c, w.act, T, c.d_ff, lng);
      RLX_LAUNCH(RLX_K_GATEUP, lng ? gemm_long_swiglu(m->w_gate_up[l], c.d_ff, d, xb, T, act, m->n_units, st)
                               : gemm_flow_swiglu_form(c.d_ff, T, m->n_units, PL, FMT)
                                   ? gemm_flow_swiglu(m->w_gate_up[l], c.d_ff, d, xb, T, act, m->n_units, st, norm_inside ? &nm : nullptr)
                                   : gemm_swiglu(m->w_gate_up[l], c.d_ff, d, xb, T, act, st));
      RLX_LAUNCH(RLX_K_DOWN, store(linear1(m->w_down[l], d, c.d_ff), act, w.planes, p_ffn));
      pend_planes = w.planes; pend_n = p_ffn.planes;
    } else {
      RLX_LAUNCH(RLX_K_ROUTER, store(linear1(m->w_router[l], c.n_experts, d), xb, w.router, p_ffn));
      RouterArgs ra = {};
      ra.logits = w.router; ra.n_planes = p_ffn.planes; ra.T = T; ra.E = c.n_experts; ra.top_k = c.top_k;
      ra.topk_idx = w.topk_idx; ra.topk_w = w.topk_w; ra.routing_out = io.out_routing; ra.layer = l;
      ra.n_layers = c.n_layers; ra.tok_live = w.meta.tok_live; ra.replay_idx = io.replay_routing;
      RLX_LAUNCH(RLX_K_GROUP, moe_route(ra, w.group_off, w.sorted_token, w.pair_pos, w.group_ws, !routed,
                                         lng ? &w.items : nullptr, st));
      const Act act = call_act(c, w.act, T * c.top_k, c.d_ff_expert, lng);
      if (lng)
        RLX_LAUNCH(RLX_K_GATEUP, gemm_long_grouped_swiglu(m->w_gate_up[l], c.d_ff_expert, d, xb, w.sorted_token, w.group_off,
                                                          act, w.items, st));
      else if (routed)
        RLX_LAUNCH(RLX_K_GATEUP, gemm_routed_swiglu(m->w_gate_up[l], c.n_experts, c.d_ff_expert, d, xb, w.topk_idx,
                                                    T * c.top_k, c.top_k, T, act, w.group_off, w.pair_pos, st));
      else
        RLX_LAUNCH(RLX_K_GATEUP, gemm_grouped_swiglu(m->w_gate_up[l], c.n_experts, c.d_ff_expert, d, xb,
                                                     w.sorted_token, w.group_off, T, T * c.top_k, act, st));
      if (lng)
        RLX_LAUNCH(RLX_K_DOWN, gemm_long_grouped_store(m->w_down[l], d, c.d_ff_expert, act, w.group_off, w.moe_y, w.items, st));
      else
        RLX_LAUNCH(RLX_K_DOWN, gemm_grouped_store(m->w_down[l], c.n_experts, d, c.d_ff_expert, act, w.group_off, T,
                                                  T * c.top_k, w.moe_y, st));
      pend_moe = true;
    }
  }

  auto lmhead = [&](const Act& x, int rows, float* logits, const uint64_t* seeds, const int32_t* sample_pos,
                    const int32_t* row_seq, bool draw, const FlowNorm* nm = nullptr) {
    if (c.n_experts == 0 && !x.pitch && gemm_flow_lmhead_form(rows, PL, FMT))
      return gemm_flow_lmhead(m->lm_head, c.vocab, d, x, rows, logits, w.lm_part, seeds, io.temperature, sample_pos, row_seq, draw, st,
                              nm);
    return x.pitch ? gemm_long_lmhead(m->lm_head, c.vocab, d, x, rows, logits, w.lm_part, seeds, io.temperature, sample_pos,
                                      row_seq, draw, m->n_units, st)
                   : gemm_lmhead(m->lm_head, c.vocab, d, x, rows, logits, w.lm_part, seeds, io.temperature, sample_pos, row_seq,
                                 draw, st);
  };

  if (io.score) {
    // every position is scored: final norm + LM head (log-sum-exp partials only, no draw) + target logit, in
    // blocks of rows; each block applies the residual still pending from the last sub-layer to its rows
    const float* pp = pend_planes; const int pn = pend_n; const bool pm = pend_moe;
    const int passes = (T + score_rows_max(T) - 1) / score_rows_max(T);
    const int per_pass = passes == 1 ? T : ((T + passes - 1) / passes + 127) / 128 * 128;   // whole token tiles
    for (int r0 = 0; r0 < T; r0 += per_pass) {
      const int n = T - r0 < per_pass ? T - r0 : per_pass;
      const Act x_lm = call_act(c, w.x_lm, n, d, rows_lmhead(c, n));
      pend_planes = pp; pend_n = pn; pend_moe = pm;
      RLX_HIP(norm(m->final_norm, w.meta.tok_iota + r0, n, x_lm, nullptr));
      RLX_LAUNCH(RLX_K_LMHEAD, lmhead(x_lm, n, nullptr, nullptr, nullptr, w.meta.tok_seq + r0, false));
      FinalizeArgs f = {};
      f.n_rows = n; f.n_parts = lmhead_parts(c.vocab, x_lm, m->n_units); f.vocab = c.vocab; f.d = d;
      f.part = w.lm_part; f.x = x_lm; f.w_lm = m->lm_head;
      f.temperature = io.temperature; f.forced = io.score_targets + r0; f.row_seq = w.meta.tok_seq + r0;
      f.eos = c.eos_token_id; f.pad = c.pad_token_id; f.out_logprobs = io.score_logprobs + r0; f.score = 1;
      RLX_HIP(sample_finalize(f, st));
    }
    return RLX_OK;
  }

  // final norm of the rows that emit a token, LM head with fused log-sum-exp / Gumbel-max partials
  const int S = io.n_seqs;
  const Act x_lm = call_act(c, w.x_lm, S, d, rows_lmhead(c, S));
  FlowNorm nm = {};
  const bool last_inside = norm_inside && io.decode;   // rows and tokens are the same (and gemm_flow_lmhead_form holds: T <= 16)
  if (last_inside) nm = inner_norm(m->final_norm);
  else RLX_HIP(norm(m->final_norm, w.meta.sample_row, S, x_lm, nullptr));
  RLX_LAUNCH(RLX_K_LMHEAD, lmhead(x_lm, S, io.out_logits, io.seeds, w.meta.sample_pos, nullptr, true, last_inside ? &nm : nullptr));
  FinalizeArgs f = {};
  f.n_rows = S; f.n_parts = lmhead_parts(c.vocab, x_lm, m->n_units); f.vocab = c.vocab; f.d = d;
  f.part = w.lm_part; f.x = x_lm; f.w_lm = m->lm_head;
  f.temperature = io.temperature; f.max_ctx_len = io.max_ctx_len; f.forced = io.forced;
  f.sample_pos = w.meta.sample_pos; f.sample_on = w.meta.sample_on;
  f.eos = c.eos_token_id; f.pad = c.pad_token_id;
  f.out_tokens = io.out_tokens; f.out_logprobs = io.out_logprobs; f.out_sampled = io.out_sampled;
  f.finished = io.finished; f.ctx_lens = io.ctx_lens_rw; f.is_decode = io.decode ? 1 : 0;
  RLX_HIP(sample_finalize(f, st));
  return RLX_OK;
}

int check_common(const rlx_model* m, const void* kv_pool, int64_t n_blocks, const void* workspace, int32_t n_seqs,
                 int32_t max_blocks_per_seq) {
  if (!m) return fail(RLX_EINVAL, "model is NULL");
  if (!kv_pool || n_blocks <= 0) return fail(RLX_EINVAL, "kv_pool is NULL or n_blocks <= 0");
  if (!workspace) return fail(RLX_EINVAL, "workspace is NULL");
  if (n_seqs < 0 || n_seqs > (1 << 16)) return fail(RLX_EINVAL, "n_seqs %d out of range", n_seqs);
  if (max_blocks_per_seq <= 0 || max_blocks_per_seq > (1 << 20))
    return fail(RLX_EINVAL, "max_blocks_per_seq %d out of range", max_blocks_per_seq);
  if (!aligned16(kv_pool) || !aligned16(workspace)) return fail(RLX_EINVAL, "kv_pool/workspace not 16-byte aligned");
  return RLX_OK;
}

// Checks a weight table against the model's shape and installs its pointers (all or nothing).
int install_weights(rlx_model* m, const rlx_weights* wt) {
  const rlx_model_config& c = m->cfg;
  const bool moe = c.n_experts > 0;
  if (wt->struct_size != sizeof(rlx_weights)) return fail(RLX_EINVAL, "rlx_weights.struct_size mismatch");
  if (!wt->embed || !wt->lm_head || !wt->final_norm) return fail(RLX_EINVAL, "NULL global weight");
  if (!aligned16(wt->embed) || !aligned16(wt->lm_head) || !aligned16(wt->final_norm))
    return fail(RLX_EINVAL, "weights must be 16-byte aligned");
  const void* const* req[] = {wt->attn_norm, wt->wq, wt->wk, wt->wv, wt->wo, wt->ffn_norm, wt->w_gate_up, wt->w_down};
  for (auto p : req)
    if (!p) return fail(RLX_EINVAL, "NULL per-layer weight table");
  if (c.qk_norm && (!wt->q_norm || !wt->k_norm)) return fail(RLX_EINVAL, "qk_norm set but q_norm/k_norm missing");
  if (moe && !wt->w_router) return fail(RLX_EINVAL, "MoE model without w_router");
  struct Table { std::vector<const h16_t*>* dst; const void* const* src; };
  std::vector<const h16_t*> t[11];
  const Table tables[11] = {
      {&m->attn_norm, wt->attn_norm}, {&m->wq, wt->wq}, {&m->wk, wt->wk}, {&m->wv, wt->wv}, {&m->wo, wt->wo},
      {&m->ffn_norm, wt->ffn_norm}, {&m->w_gate_up, wt->w_gate_up}, {&m->w_down, wt->w_down},
      {&m->q_norm, c.qk_norm ? wt->q_norm : nullptr}, {&m->k_norm, c.qk_norm ? wt->k_norm : nullptr},
      {&m->w_router, moe ? wt->w_router : nullptr}};
  for (int i = 0; i < 11; ++i) {
    t[i].assign(c.n_layers, nullptr);
    if (!tables[i].src) continue;
    for (int l = 0; l < c.n_layers; ++l) {
      if (!tables[i].src[l] || !aligned16(tables[i].src[l]))
        return fail(RLX_EINVAL, "a per-layer weight pointer is NULL or not 16-byte aligned");
      t[i][l] = (const h16_t*)tables[i].src[l];
    }
  }
  for (int i = 0; i < 11; ++i) tables[i].dst->swap(t[i]);
  m->embed = (const h16_t*)wt->embed; m->lm_head = (const h16_t*)wt->lm_head;
  m->final_norm = (const h16_t*)wt->final_norm;
  return RLX_OK;
}

int decode_step(const rlx_model* m, void* kv_pool, int64_t n_blocks, void* workspace, size_t workspace_bytes, int32_t n_seqs,
                int32_t* tokens_inout, int32_t* ctx_lens_inout, const int32_t* block_table, int32_t max_blocks_per_seq,
                const uint64_t* seeds, const float* temperature, const int32_t* max_ctx_len, uint8_t* finished_inout,
                const int32_t* forced_tokens, float* out_logprobs, int32_t* out_sampled, int32_t* out_routing,
                float* out_logits, const void* shared_prefix, bool lean, void* stream) {
  int rc = check_common(m, kv_pool, n_blocks, workspace, n_seqs, max_blocks_per_seq);
  if (rc) return rc;
  if (n_seqs == 0) return RLX_OK;                         // an empty step: nothing to enqueue, no array is read
  if (!tokens_inout || !ctx_lens_inout || !block_table || !seeds || !temperature || !max_ctx_len ||
      !finished_inout || !out_logprobs)
    return fail(RLX_EINVAL, "NULL array argument");
  if (shared_prefix && !aligned16(shared_prefix)) return fail(RLX_EINVAL, "shared_prefix must be 16-byte aligned");
  Workspace w = carve(m->cfg, (char*)workspace, n_seqs, n_seqs, call_planes(m->cfg, n_seqs, lean));
  if (w.bytes > workspace_bytes)
    return fail(RLX_ENOMEM, "workspace too small: need %zu bytes, have %zu", w.bytes, workspace_bytes);
  hipStream_t st = (hipStream_t)stream;
  DecodeBeginArgs b = {};
  b.n_seqs = n_seqs; b.Hkv = m->cfg.n_kv_heads; b.head_dim = m->cfg.head_dim;
  b.ctx_lens = ctx_lens_inout; b.finished = finished_inout; b.block_table = block_table; b.max_blocks = max_blocks_per_seq;
  b.meta = w.meta; b.inv_freq = m->inv_freq;
  b.embed = m->embed; b.vocab = m->cfg.vocab; b.d_model = m->cfg.d_model; b.dtype = m->cfg.dtype;
  b.tokens = tokens_inout; b.h = w.h;
  b.team = attn_by_team(m->cfg); b.shared = (const int32_t*)shared_prefix;
  b.unit_prefix = w.attn_prefix; b.share_start = w.attn_share_start; b.plan_hdr = w.attn_hdr;
  RLX_HIP(decode_begin(b, m->attn_wgs, st));
  StepIO io = {};
  io.n_seqs = n_seqs; io.T = n_seqs; io.decode = true;
  io.tokens = tokens_inout; io.ctx_lens = ctx_lens_inout; io.ctx_lens_rw = ctx_lens_inout;
  io.block_table = block_table; io.max_blocks = max_blocks_per_seq;
  io.seeds = seeds; io.temperature = temperature; io.max_ctx_len = max_ctx_len; io.forced = forced_tokens;
  io.out_tokens = tokens_inout; io.out_logprobs = out_logprobs; io.finished = finished_inout;
  io.out_sampled = out_sampled; io.out_routing = m->cfg.n_experts ? out_routing : nullptr; io.out_logits = out_logits;
  io.shared_prefix = (const int32_t*)shared_prefix; io.lean = lean;
  return run_layers(m, (h16_t*)kv_pool, n_blocks, w, io, st);
}

}  // namespace

extern "C" {

const char* rlx_last_error(void) { return g_err; }

int rlx_model_create(const rlx_model_config* cfg, const rlx_weights* wt, rlx_model** out) {
  if (!cfg || !wt || !out) return fail(RLX_EINVAL, "NULL argument");
  *out = nullptr;
  if (cfg->struct_size != sizeof(rlx_model_config)) return fail(RLX_EINVAL, "rlx_model_config.struct_size mismatch");
  const rlx_model_config& c = *cfg;
  if (c.n_layers <= 0 || c.d_model <= 0 || c.n_q_heads <= 0 || c.n_kv_heads <= 0 || c.vocab <= 0)
    return fail(RLX_EINVAL, "non-positive dimension");
  if (c.head_dim != 64 && c.head_dim != 128) return fail(RLX_EUNSUPPORTED, "head_dim %d (64 or 128)", c.head_dim);
  if (c.kv_block_size != 16) return fail(RLX_EUNSUPPORTED, "kv_block_size %d (must be 16)", c.kv_block_size);
  if (c.n_q_heads % c.n_kv_heads) return fail(RLX_EINVAL, "n_q_heads not a multiple of n_kv_heads");
  if (c.n_q_heads / c.n_kv_heads > 16) return fail(RLX_EUNSUPPORTED, "GQA group > 16");
  if (c.d_model % 16) return fail(RLX_EUNSUPPORTED, "d_model must be a multiple of 16");
  const bool moe = c.n_experts > 0;
  if (moe) {
    if (c.n_experts > 256 || c.top_k <= 0 || c.top_k > 8 || c.top_k > c.n_experts || c.d_ff_expert <= 0)
      return fail(RLX_EUNSUPPORTED, "MoE limits: n_experts <= 256, 1 <= top_k <= min(8, n_experts)");
    if (c.d_ff_expert % 16 || c.d_ff) return fail(RLX_EINVAL, "MoE: d_ff_expert %% 16 == 0 and d_ff == 0 required");
  } else {
    if (c.d_ff <= 0 || c.d_ff % 16) return fail(RLX_EINVAL, "dense: d_ff must be a positive multiple of 16");
    if (c.top_k || c.d_ff_expert) return fail(RLX_EINVAL, "dense: top_k and d_ff_expert must be 0");
  }
  if (c.eos_token_id < 0 || c.eos_token_id >= c.vocab || c.pad_token_id < 0 || c.pad_token_id >= c.vocab)
    return fail(RLX_EINVAL, "eos/pad token id outside the vocabulary");
  if (!(c.rms_eps >= 0.f) || !(c.rope_theta > 0.f)) return fail(RLX_EINVAL, "rms_eps / rope_theta");
  if (c.activation_split != 0 && c.activation_split != 1) return fail(RLX_EINVAL, "activation_split must be 0 or 1");
  if (c.qk_norm != 0 && c.qk_norm != 1) return fail(RLX_EINVAL, "qk_norm must be 0 or 1");
  if (c.dtype != RLX_DTYPE_BF16 && c.dtype != RLX_DTYPE_F16) return fail(RLX_EINVAL, "dtype must be RLX_DTYPE_BF16 or RLX_DTYPE_F16");
  if (c.dtype == RLX_DTYPE_F16 && c.activation_split)
    return fail(RLX_EUNSUPPORTED, "fp16 models carry activations as one term: activation_split must be 0");

  rlx_model* m = new (std::nothrow) rlx_model();
  if (!m) return fail(RLX_ENOMEM, "host allocation failed");
  m->cfg = c;
  m->inv_freq = nullptr;
  m->static_ws = nullptr;
  m->weight_version = 0;
  const int rc = install_weights(m, wt);
  if (rc != RLX_OK) {
    delete m;
    return rc;
  }
  // rotary frequencies theta^(-2i/hd) in double
  std::vector<double> inv(c.head_dim / 2);
  for (int i = 0; i < c.head_dim / 2; ++i) inv[i] = pow((double)c.rope_theta, -2.0 * i / c.head_dim);
  hipError_t e = hipGetDevice(&m->device);
  int n_cu = 0;
  if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, m->device);
  m->n_units = n_cu > 0 ? n_cu : 1;
  gemm_set_units(m->n_units);
  m->attn_wgs = 2 * n_cu < ATTN_WGS_MAX ? (2 * n_cu > 0 ? 2 * n_cu : 1) : ATTN_WGS_MAX;
  if (e == hipSuccess && scratch_on_device(m->device, &m->static_ws) != hipSuccess) {
    // checked, not fatal: the model works with caller workspaces; rollout_decode_step_static reports the missing array
    m->static_ws = nullptr;
    (void)hipGetLastError();
  }
  if (e == hipSuccess) e = hipMalloc((void**)&m->inv_freq, inv.size() * sizeof(double));
  if (e == hipSuccess) e = hipMemcpy(m->inv_freq, inv.data(), inv.size() * sizeof(double), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    if (m->inv_freq) (void)hipFree(m->inv_freq);
    delete m;
    return fail(RLX_EHIP, "rlx_model_create: %s", hipGetErrorString(e));
  }
  *out = m;
  return RLX_OK;
}

int rlx_model_set_attention_grid(rlx_model* m, int32_t n_workgroups) {
  if (!m) return fail(RLX_EINVAL, "model is NULL");
  if (n_workgroups < 1 || n_workgroups > ATTN_WGS_MAX)
    return fail(RLX_EINVAL, "rlx_model_set_attention_grid: n_workgroups %d outside 1..%d", n_workgroups, ATTN_WGS_MAX);
  m->attn_wgs = n_workgroups;
  return RLX_OK;
}

int rlx_model_set_weights(rlx_model* m, const rlx_weights* w, uint64_t version) {
  if (!m || !w) return fail(RLX_EINVAL, "rlx_model_set_weights: NULL argument");
  const int rc = install_weights(m, w);
  if (rc == RLX_OK) m->weight_version = version;
  return rc;
}

int rlx_model_weight_version(const rlx_model* m, uint64_t* version_out) {
  if (!m || !version_out) return fail(RLX_EINVAL, "rlx_model_weight_version: NULL argument");
  *version_out = m->weight_version;
  return RLX_OK;
}

int rlx_model_destroy(rlx_model* m) {
  if (!m) return RLX_OK;
  hipError_t e = m->inv_freq ? hipFree(m->inv_freq) : hipSuccess;
  delete m;
  if (e != hipSuccess) return fail(RLX_EHIP, "hipFree: %s", hipGetErrorString(e));
  return RLX_OK;
}

int rlx_kv_pool_bytes(const rlx_model* m, int64_t n_blocks, size_t* bytes_out) {
  if (!m || !bytes_out || n_blocks <= 0) return fail(RLX_EINVAL, "bad argument");
  *bytes_out = (size_t)m->cfg.n_layers * (size_t)n_blocks * block_elems(m->cfg) * 2;
  return RLX_OK;
}

int rlx_workspace_bytes(const rlx_model* m, int32_t max_seqs, int32_t max_tokens, int32_t max_blocks_per_seq,
                        size_t* bytes_out) {
  if (!m || !bytes_out || max_seqs <= 0 || max_tokens < max_seqs || max_blocks_per_seq <= 0)
    return fail(RLX_EINVAL, "bad argument (need 0 < max_seqs <= max_tokens, max_blocks_per_seq > 0)");
  const PlaneRows planes = {plane_rows_up_to(m->cfg, max_tokens, false), plane_rows_up_to(m->cfg, max_tokens, true)};
  const size_t b = carve(m->cfg, nullptr, max_seqs, max_tokens, planes).bytes;   // no buffer gets smaller as a call grows
  *bytes_out = b;
  return RLX_OK;
}

int rlx_kv_copy_blocks(const rlx_model* m, void* kv_pool, int64_t n_blocks, const int32_t* src, const int32_t* dst,
                       int32_t n, void* stream) {
  if (!m || !kv_pool || n_blocks <= 0 || n < 0 || (n > 0 && (!src || !dst))) return fail(RLX_EINVAL, "bad argument");
  RLX_HIP(kv_copy_blocks((h16_t*)kv_pool, n_blocks, m->cfg.n_layers, block_elems(m->cfg), src, dst, n,
                         (hipStream_t)stream));
  return RLX_OK;
}

int rollout_prefill_chunk(const rlx_model* m, void* kv_pool, int64_t n_blocks, void* workspace, size_t workspace_bytes,
                          int32_t n_seqs, int32_t total_tokens, const int32_t* token_ids, const void* input_embeds,
                          const int32_t* cu_seqlens, const int32_t* ctx_lens, const int32_t* block_table,
                          int32_t max_blocks_per_seq, const uint8_t* sample_last, const uint64_t* seeds,
                          const float* temperature, const int32_t* max_ctx_len, const int32_t* forced_tokens,
                          int32_t* out_tokens, float* out_logprobs, uint8_t* finished_out, int32_t* out_sampled,
                          int32_t* out_routing, float* out_logits, void* stream) {
  int rc = check_common(m, kv_pool, n_blocks, workspace, n_seqs, max_blocks_per_seq);
  if (rc) return rc;
  if (n_seqs == 0 && total_tokens == 0) return RLX_OK;   // an empty call: nothing to enqueue, no array is read
  if (n_seqs == 0 || total_tokens <= 0 || total_tokens > (1 << 24))
    return fail(RLX_EINVAL, "total_tokens %d out of range for %d sequences", total_tokens, n_seqs);
  if (!token_ids || !cu_seqlens || !ctx_lens || !block_table || !sample_last || !seeds || !temperature ||
      !max_ctx_len || !out_tokens || !out_logprobs || !finished_out)
    return fail(RLX_EINVAL, "NULL array argument");
  if (input_embeds && !aligned16(input_embeds)) return fail(RLX_EINVAL, "input_embeds not 16-byte aligned");
  const int T = total_tokens > n_seqs ? total_tokens : n_seqs;
  Workspace w = carve(m->cfg, (char*)workspace, n_seqs, T, call_planes(m->cfg, total_tokens));
  if (w.bytes > workspace_bytes)
    return fail(RLX_ENOMEM, "workspace too small: need %zu bytes, have %zu", w.bytes, workspace_bytes);
  hipStream_t st = (hipStream_t)stream;
  RLX_HIP(meta_prefill(w.meta, n_seqs, total_tokens, cu_seqlens, ctx_lens, sample_last, m->inv_freq, m->cfg.head_dim, st));
  StepIO io = {};
  io.n_seqs = n_seqs; io.T = total_tokens; io.decode = false;
  io.tokens = token_ids; io.input_embeds = (const h16_t*)input_embeds; io.cu_seqlens = cu_seqlens;
  io.ctx_lens = ctx_lens; io.block_table = block_table; io.max_blocks = max_blocks_per_seq;
  io.seeds = seeds; io.temperature = temperature; io.max_ctx_len = max_ctx_len; io.forced = forced_tokens;
  io.out_tokens = out_tokens; io.out_logprobs = out_logprobs; io.finished = finished_out;
  io.out_sampled = out_sampled; io.out_routing = m->cfg.n_experts ? out_routing : nullptr; io.out_logits = out_logits;
  return run_layers(m, (h16_t*)kv_pool, n_blocks, w, io, st);
}

int rollout_score_chunk(const rlx_model* m, void* kv_pool, int64_t n_blocks, void* workspace, size_t workspace_bytes,
                        int32_t n_seqs, int32_t total_tokens, const int32_t* token_ids, const void* input_embeds,
                        const int32_t* cu_seqlens, const int32_t* ctx_lens, const int32_t* block_table,
                        int32_t max_blocks_per_seq, const int32_t* target_ids, const float* temperature,
                        const int32_t* replay_routing, float* out_logprobs, int32_t* out_routing, void* stream) {
  int rc = check_common(m, kv_pool, n_blocks, workspace, n_seqs, max_blocks_per_seq);
  if (rc) return rc;
  if (n_seqs == 0 && total_tokens == 0) return RLX_OK;   // an empty call: nothing to enqueue, no array is read
  if (n_seqs == 0 || total_tokens <= 0 || total_tokens > (1 << 24))
    return fail(RLX_EINVAL, "total_tokens %d out of range for %d sequences", total_tokens, n_seqs);
  if (!token_ids || !cu_seqlens || !ctx_lens || !block_table || !target_ids || !temperature || !out_logprobs)
    return fail(RLX_EINVAL, "NULL array argument");
  if (input_embeds && !aligned16(input_embeds)) return fail(RLX_EINVAL, "input_embeds not 16-byte aligned");
  const int T = total_tokens > n_seqs ? total_tokens : n_seqs;
  Workspace w = carve(m->cfg, (char*)workspace, n_seqs, T, call_planes(m->cfg, total_tokens));
  if (w.bytes > workspace_bytes)
    return fail(RLX_ENOMEM, "workspace too small: need %zu bytes, have %zu", w.bytes, workspace_bytes);
  hipStream_t st = (hipStream_t)stream;
  RLX_HIP(meta_prefill(w.meta, n_seqs, total_tokens, cu_seqlens, ctx_lens, nullptr, m->inv_freq, m->cfg.head_dim, st));
  StepIO io = {};
  io.n_seqs = n_seqs; io.T = total_tokens; io.decode = false;
  io.tokens = token_ids; io.input_embeds = (const h16_t*)input_embeds; io.cu_seqlens = cu_seqlens;
  io.ctx_lens = ctx_lens; io.block_table = block_table; io.max_blocks = max_blocks_per_seq;
  io.temperature = temperature;
  io.out_routing = m->cfg.n_experts ? out_routing : nullptr;
  io.score = true; io.score_targets = target_ids; io.score_logprobs = out_logprobs;
  io.replay_routing = m->cfg.n_experts ? replay_routing : nullptr;
  return run_layers(m, (h16_t*)kv_pool, n_blocks, w, io, st);
}

int rollout_decode_step_shared(const rlx_model* m, void* kv_pool, int64_t n_blocks, void* workspace,
                               size_t workspace_bytes, int32_t n_seqs, int32_t* tokens_inout, int32_t* ctx_lens_inout,
                               const int32_t* block_table, int32_t max_blocks_per_seq, const uint64_t* seeds,
                               const float* temperature, const int32_t* max_ctx_len, uint8_t* finished_inout,
                               const int32_t* forced_tokens, float* out_logprobs, int32_t* out_sampled,
                               int32_t* out_routing, float* out_logits, const void* shared_prefix, void* stream) {
  return decode_step(m, kv_pool, n_blocks, workspace, workspace_bytes, n_seqs, tokens_inout, ctx_lens_inout, block_table,
                     max_blocks_per_seq, seeds, temperature, max_ctx_len, finished_inout, forced_tokens, out_logprobs,
                     out_sampled, out_routing, out_logits, shared_prefix, false, stream);
}

int rollout_decode_step(const rlx_model* m, void* kv_pool, int64_t n_blocks, void* workspace, size_t workspace_bytes,
                        int32_t n_seqs, int32_t* tokens_inout, int32_t* ctx_lens_inout, const int32_t* block_table,
                        int32_t max_blocks_per_seq, const uint64_t* seeds, const float* temperature,
                        const int32_t* max_ctx_len, uint8_t* finished_inout, const int32_t* forced_tokens,
                        float* out_logprobs, int32_t* out_sampled, int32_t* out_routing, float* out_logits,
                        void* stream) {
  return rollout_decode_step_shared(m, kv_pool, n_blocks, workspace, workspace_bytes, n_seqs, tokens_inout,
                                    ctx_lens_inout, block_table, max_blocks_per_seq, seeds, temperature, max_ctx_len,
                                    finished_inout, forced_tokens, out_logprobs, out_sampled, out_routing, out_logits,
                                    nullptr, stream);
}

int rollout_decode_step_static(const rlx_model* m, void* kv_pool, int64_t n_blocks, int32_t n_seqs,
                               int32_t* tokens_inout, int32_t* ctx_lens_inout, const int32_t* block_table,
                               int32_t max_blocks_per_seq, const uint64_t* seeds, const float* temperature,
                               const int32_t* max_ctx_len, uint8_t* finished_inout, const int32_t* forced_tokens,
                               float* out_logprobs, int32_t* out_sampled, int32_t* out_routing, float* out_logits,
                               void* stream) {
  if (!m) return fail(RLX_EINVAL, "model is NULL");
  if (n_seqs < 0 || n_seqs > (1 << 16)) return fail(RLX_EINVAL, "n_seqs %d out of range", n_seqs);
  if (max_blocks_per_seq <= 0 || max_blocks_per_seq > (1 << 20))
    return fail(RLX_EINVAL, "max_blocks_per_seq %d out of range", max_blocks_per_seq);
  size_t need = n_seqs ? carve(m->cfg, nullptr, n_seqs, n_seqs, call_planes(m->cfg, n_seqs)).bytes : 0;
  const bool lean = need > (size_t)RLX_STATIC_WORKSPACE_BYTES;
  if (lean) need = carve(m->cfg, nullptr, n_seqs, n_seqs, call_planes(m->cfg, n_seqs, true)).bytes;
  if (need > (size_t)RLX_STATIC_WORKSPACE_BYTES)
    return fail(RLX_ENOMEM, "rollout_decode_step_static: a step of %d sequences of this model needs %zu bytes of "
                "scratch, the fixed array holds %zu; use rollout_decode_step with a workspace of your own", n_seqs,
                need, (size_t)RLX_STATIC_WORKSPACE_BYTES);
  if (!m->static_ws) return fail(RLX_EHIP, "rollout_decode_step_static: the fixed scratch array has no address");
  return decode_step(m, kv_pool, n_blocks, m->static_ws, (size_t)RLX_STATIC_WORKSPACE_BYTES, n_seqs, tokens_inout,
                     ctx_lens_inout, block_table, max_blocks_per_seq, seeds, temperature, max_ctx_len, finished_inout,
                     forced_tokens, out_logprobs, out_sampled, out_routing, out_logits, nullptr, lean, stream);
}

int rlx_shared_prefix_bytes(const rlx_model* m, int32_t n_seqs, size_t* bytes_out) {
  if (!m || !bytes_out || n_seqs <= 0 || n_seqs > (1 << 16)) return fail(RLX_EINVAL, "rlx_shared_prefix_bytes: bad argument");
  *bytes_out = align_up(shared_prefix_words(n_seqs, m->cfg.n_kv_heads) * 4);
  return RLX_OK;
}

int rlx_shared_prefix_build(const rlx_model* m, int32_t n_seqs, const int32_t* leader, const int32_t* shared_pages,
                            void* desc, size_t desc_bytes, void* stream) {
  if (!m || !leader || !shared_pages || !desc || n_seqs <= 0 || n_seqs > (1 << 16))
    return fail(RLX_EINVAL, "rlx_shared_prefix_build: bad argument");
  if (!aligned16(desc)) return fail(RLX_EINVAL, "rlx_shared_prefix_build: desc must be 16-byte aligned");
  const size_t words = shared_prefix_words(n_seqs, m->cfg.n_kv_heads);
  if (desc_bytes < words * 4) return fail(RLX_ENOMEM, "rlx_shared_prefix_build: desc needs %zu bytes", words * 4);
  for (int i = 0; i < n_seqs; ++i)
    if (leader[i] < 0 || leader[i] > i || shared_pages[i] < 0)
      return fail(RLX_EINVAL, "rlx_shared_prefix_build: sequence %d: leader %d (0..%d) / shared_pages %d", i, leader[i],
                  i, shared_pages[i]);
  std::vector<int32_t> host;
  try {                                               // the groups' list and the staging copy: no exception leaves a C entry
    host.resize(words);
    // MoE policies keep the order of their sums: the same chunks however many tiles that makes
    shared_prefix_build(n_seqs, m->cfg.n_q_heads, m->cfg.n_kv_heads, leader, shared_pages, attn_by_team(m->cfg) ? 0 : prefix_wgs(m),
                        shared_prefix_plain_units(m->cfg.head_dim, m->cfg.n_layers), host.data());
  } catch (const std::bad_alloc&) {
    return fail(RLX_ENOMEM, "rlx_shared_prefix_build: host allocation failed");
  }
  hipStream_t st = (hipStream_t)stream;
  RLX_HIP(hipMemcpyAsync(desc, host.data(), words * 4, hipMemcpyHostToDevice, st));
  RLX_HIP(hipStreamSynchronize(st));      // the staging vector dies with this call
  return RLX_OK;
}

int rlx_profile_kernel(int32_t kernel_class, void* const* start_events, void* const* stop_events, int32_t n_events,
                       int32_t stride) {
  if (kernel_class == 0 || n_events <= 0) {
    int used = g_prof.used;
    g_prof = ProfState();
    return used;
  }
  if (!start_events || !stop_events || stride <= 0 || kernel_class < 0 || kernel_class > RLX_K_ATTN_PREFIX)
    return fail(RLX_EINVAL, "rlx_profile_kernel: bad argument");
  g_prof = ProfState();
  g_prof.cls = kernel_class; g_prof.start = start_events; g_prof.stop = stop_events; g_prof.n = n_events;
  g_prof.stride = stride;
  return 0;
}

int rlx_packed_weight_bytes(int32_t n, int32_t k, size_t* bytes_out) {
  if (!bytes_out || n <= 0 || k <= 0 || (k % 16)) return fail(RLX_EINVAL, "rlx_packed_weight_bytes: k %% 16 == 0 required");
  *bytes_out = packed_weight_elems(n, k) * 2;
  return RLX_OK;
}

int rlx_pack_weight(const void* src, void* dst, int32_t count, int32_t n, int32_t k, void* stream) {
  if (!src || !dst || count <= 0 || n <= 0 || k <= 0 || (k % 16))
    return fail(RLX_EINVAL, "rlx_pack_weight: bad argument (k %% 16 == 0 required)");
  if (!aligned16(src) || !aligned16(dst)) return fail(RLX_EINVAL, "rlx_pack_weight: 16-byte alignment");
  const size_t pe = packed_weight_elems(n, k);
  for (int i = 0; i < count; ++i)
    RLX_HIP(pack_weight((const h16_t*)src + (size_t)i * n * k, (h16_t*)dst + (size_t)i * pe, n, k,
                        (hipStream_t)stream));
  return RLX_OK;
}

int rlx_pack_gate_up(const void* gate, const void* up, void* dst, int32_t count, int32_t f, int32_t k, void* stream) {
  if (!gate || !up || !dst || count <= 0 || f <= 0 || k <= 0 || (k % 16) || (f % 16))
    return fail(RLX_EINVAL, "rlx_pack_gate_up: bad argument (f %% 16 == 0 and k %% 16 == 0 required)");
  if (!aligned16(gate) || !aligned16(up) || !aligned16(dst)) return fail(RLX_EINVAL, "rlx_pack_gate_up: 16-byte alignment");
  const size_t pe = packed_weight_elems(2 * f, k);
  for (int i = 0; i < count; ++i)
    RLX_HIP(pack_gate_up((const h16_t*)gate + (size_t)i * f * k, (const h16_t*)up + (size_t)i * f * k,
                         (h16_t*)dst + (size_t)i * pe, f, k, (hipStream_t)stream));
  return RLX_OK;
}

int rlx_op_linear(const void* x, const void* w, float* y, int32_t n_tokens, int32_t n, int32_t k, void* workspace,
                  size_t workspace_bytes, void* stream) {
  if (!x || !w || !y || n_tokens <= 0 || n <= 0 || k <= 0 || (k % 16) || (n % 4))
    return fail(RLX_EINVAL, "rlx_op_linear: bad argument (k %% 16 == 0, n %% 4 == 0 required)");
  if (!aligned16(x) || !aligned16(w) || !aligned16(y) || !workspace || !aligned16(workspace))
    return fail(RLX_EINVAL, "rlx_op_linear: NULL workspace or 16-byte alignment");
  int dev = 0, n_units = 0;
  RLX_HIP(hipGetDevice(&dev));
  RLX_HIP(hipDeviceGetAttribute(&n_units, hipDeviceAttributeMultiprocessorCount, dev));
  const int splits = n_tokens <= 256 ? gemm_plan_splits(n, k, n_tokens, gemm_max_splits(), n_units > 0 ? n_units : 1, 1, DT_BF16) : 1;
  hipStream_t st = (hipStream_t)stream;
  const size_t xb = align_up(frag_act_elems(n_tokens, k, 1) * 2);
  const size_t pb = splits > 1 ? align_up((size_t)splits * n_tokens * n * 4) : 0;
  if (workspace_bytes < xb + pb) return fail(RLX_ENOMEM, "rlx_op_linear: workspace needs %zu bytes", xb + pb);
  h16_t* xp = (h16_t*)workspace;
  float* planes = (float*)((char*)workspace + xb);
  RLX_HIP(pack_activation((const h16_t*)x, xp, n_tokens, k, st));
  const Act xa = make_act(xp, n_tokens, k, 1, DT_BF16);
  if (splits == 1) {
    RLX_HIP(gemm_store(linear1(w, n, k), xa, n_tokens, y, n, 1, st));
    return RLX_OK;
  }
  RLX_HIP(gemm_store(linear1(w, n, k), xa, n_tokens, planes, n, splits, st));
  RLX_HIP(sum_planes(planes, splits, (size_t)n_tokens * n, y, st));
  return RLX_OK;
}

}  // extern "C"
