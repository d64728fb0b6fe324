// Weight-streaming skinny GEMM for decode and chunked prefill (gfx950, MFMA 32x32x16 on bf16 or fp16 operands).
//
//   y[t, n] = sum_k x[t, k] * W[n, k]        fp32 accumulate
//
// Both operands are stored in MFMA fragment order (see common.h): every weight load of a wave
// reads one 1 KB block, eight full cache lines, nothing wasted, and the texture-address path is
// left free for the activations; the blocks of the four tiles of a workgroup alternate along k,
// so the workgroup as a whole streams one contiguous run.
// Each of the four waves of a workgroup owns one 32-row tile of W over the
// workgroup's K range and keeps two batches of weight fragments in flight in registers
// (HBM latency under load is several microseconds, so the bytes in flight per CU decide
// the achieved bandwidth).  The activations of the current K chunk are shared by the four
// waves through LDS (double buffered); the next chunk is fetched while the current one is
// multiplied.  No reduction across waves is needed.  Optional split-K across workgroups
// writes partial planes that the consumer adds in plane order (deterministic).
//
// Epilogues: plain store (q|k|v, o and down projections, expert down projection),
// SwiGLU (gate/up), LM head with fused log-sum-exp and Gumbel-max partials per 32-row tile.
#include <math.h>

#include <atomic>
#include <mutex>

#include "gemm_core.h"

namespace rlx {

namespace {

constexpr int GEMM_WAVES = 4;
constexpr int GEMM_THREADS = GEMM_WAVES * WAVE;

template <int MT, int PL>
struct Tiling {
  // k-steps per LDS chunk: 32 fragments (64 KB for both buffers) in general.  The 32-token two-term form, which
  // the expert-grouped decode GEMMs launch as thousands of workgroups, takes 24 (48 KB): with 64 KB only one
  // workgroup was resident per compute unit (in-kernel timestamps), with 48 KB two are (expert down GEMM -6 %).
  static constexpr int KC = (MT == 1 && PL == 2) ? 12 : ((32 / (MT * PL)) > 16 ? 16 : (32 / (MT * PL)));
  static constexpr int U = KC / 2;                                          // k-steps per weight batch (store form)
  static constexpr int FRAGS = KC * MT * PL;                                // 1 KB fragments per chunk
  static constexpr int PER_THREAD = FRAGS / GEMM_WAVES;                     // staged by each wave
  static constexpr int LDS_BYTES = 2 * FRAGS * 1024;
  static_assert(LDS_BYTES >= GEMM_WAVES * 4 * 1024, "the LM-head epilogue's scratch fits");
};

// ONCE: the launch reads every weight once (a single token tile per weight tile), so the weight loads are marked
// non-temporal; with several token tiles the later ones find the weights in the caches, and the mark would send
// them to memory again (decode steps of 129..256 tokens: down projection +10 % with the mark).
// at least two waves per SIMD: beyond 256 registers only one workgroup would be resident per unit
template <int MT, int EPI, int PL, int FMT, bool ONCE>
__global__ __launch_bounds__(GEMM_THREADS, 2) void gemm_skinny_kernel(GemmArgs a) {
  using TL = Tiling<MT, PL>;
  constexpr int KC = TL::KC, U = TL::U, FRAGS = TL::FRAGS, PT = TL::PER_THREAD;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  u32x4* lds = reinterpret_cast<u32x4*>(lds_raw);   // [2][FRAGS][64 lanes]

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r32 = lane & 31, half = lane >> 5;
  const int mt0 = blockIdx.z * MT;                  // first 32-token tile of this workgroup
  int split = blockIdx.y;
  int row_base = 0;
  const bool grouped = a.group_off != nullptr;
  if (grouped) {
    const int e = blockIdx.y;
    row_base = a.group_off[e];
    a.T = a.group_off[e + 1] - row_base;
    if (mt0 * 32 >= a.T) return;                    // uniform over the workgroup, before any barrier
    a.w[0] += (size_t)e * a.w_expert_stride;
    split = 0;
  }

  // ---- this wave's weight tile ----
  // Every load below is unconditional (clamped address) and masked afterwards, so the main loop is
  // straight-line code and the hardware counters, not branches, order loads against their uses.
  const int KS = a.K >> 4;
  const int n_tiles = (a.N + 31) >> 5;
  const int nt = blockIdx.x * GEMM_WAVES + wave;
  const bool have_tile = nt < n_tiles;
  const h16_t* wp;
  {
    int lt = have_tile ? nt : 0;                    // a wave without a tile re-reads tile 0 and stores nothing
    const h16_t* base = a.w[0];                    // static member picks keep the pointers in the global space
    if (lt >= a.w_tiles[0]) {
      lt -= a.w_tiles[0];
      base = a.w[1];
      if (lt >= a.w_tiles[1]) { lt -= a.w_tiles[1]; base = a.w[2]; }
    }
    wp = base + packed_tile_offset(lt, KS) + lane * 8;
  }
  const int ks_b = split * a.ksteps_per_split;
  int ks_e = ks_b + a.ksteps_per_split;
  if (ks_e > KS) ks_e = KS;                          // the host never launches an empty split

  // ---- activation staging: each wave moves PT fragments of a chunk ----
  // fragment f of a chunk = (k-step f / (MT*PL), token tile (f / PL) % MT, plane f % PL)
  const h16_t* xsrc[MT];
  bool xok[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    if (grouped) {
      const int r = (mt0 + m) * 32 + r32;
      xok[m] = r < a.T;
      const int rr = xok[m] ? r : 0;
      const int row = a.x_rows ? a.x_rows[row_base + rr] : row_base + rr;
      xsrc[m] = a.x + frag_act_offset(row, 8 * half, 0, a.x_mtiles, PL);
    } else {
      xok[m] = mt0 + m < a.x_mtiles;
      const int mt = xok[m] ? mt0 + m : 0;
      xsrc[m] = a.x + (size_t)mt * PL * 512 + lane * 8;
    }
  }
  const size_t x_kstride = (size_t)a.x_mtiles * PL * 512;   // elements between consecutive k-steps
  // factor the norm left to this kernel's outputs (Act::ss), or 1: the sums are requested first of all, so that
  // no later wait has to sit through the weight batches for them, and turned into the factor after the first barrier
  f32x4 ssq[MT];
  float rs[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int t = (mt0 + m) * 32 + r32;
    ssq[m] = f32x4{1.f, 1.f, 1.f, 1.f};
    if (a.x_ss && !grouped) ssq[m] = row_ss(a, t < a.T ? t : 0);
  }
  LmRow lm[MT];                                       // LM head: likewise requested first of all ...
  auto fetch_lm_rows = [&]() {
#pragma unroll
    for (int m = 0; m < MT; ++m)
      if constexpr (EPI == EPI_LMHEAD) lm[m] = lm_row(a, (mt0 + m) * 32 + r32);
  };
  if (PL == 2) fetch_lm_rows();                       // ... or last, where 256 registers are taken without them
  __builtin_amdgcn_sched_barrier(0);
  // Fragment i of this wave belongs to the same token tile in every chunk.  With four token tiles the tile is picked
  // here, once, by comparing the wave number with constants, so that the arrays above are only ever indexed by
  // constants: the compiler turned the run-time choice among four into an indexed access, which put the arrays
  // into scratch memory with loads from it in the main loop (with two tiles it selects, in fewer registers).
  constexpr int NSEL = MT == 4 ? PT : 1;
  const h16_t* xsel[NSEL];
  bool oksel[NSEL];
  if (MT == 4) {
#pragma unroll
    for (int i = 0; i < NSEL; ++i) {
      xsel[i] = xsrc[0];
      oksel[i] = xok[0];
#pragma unroll
      for (int w = 0; w < GEMM_WAVES; ++w) {
        const int mw = ((w + GEMM_WAVES * i) / PL) % MT;      // a constant once both loops are unrolled
        if (wave == w) { xsel[i] = xsrc[mw]; oksel[i] = xok[mw]; }
      }
    }
  }
  auto tile_of = [&](int i, const h16_t*& src, bool& ok) {
    if (MT == 4) { src = xsel[i]; ok = oksel[i]; return; }
    const int m = ((wave + GEMM_WAVES * i) / PL) % MT;
    src = xsrc[0]; ok = xok[0];
#pragma unroll
    for (int mm = 1; mm < MT; ++mm)
      if (m == mm) { src = xsrc[mm]; ok = xok[mm]; }
  };
  auto stage_load = [&](int chunk, u32x4 (&r)[PT]) {
    const int ks0 = ks_b + chunk * KC;
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int f = wave + GEMM_WAVES * i;
      const int ks = ks0 + f / (MT * PL), p = f % PL;
      const int ksc = ks < ks_e ? ks : ks_e - 1;
      const h16_t* src;
      bool ok;
      tile_of(i, src, ok);
      (void)ok;
      r[i] = *reinterpret_cast<const u32x4*>(src + (size_t)ksc * x_kstride + (size_t)p * 512);
    }
  };
  // the mask is applied when the fragments are written to LDS, long after the loads were issued
  auto stage_store = [&](int chunk, const u32x4 (&r)[PT]) {
    const int ks0 = ks_b + chunk * KC;
    const int buf = chunk & 1;
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int f = wave + GEMM_WAVES * i;
      const int ks = ks0 + f / (MT * PL);
      const h16_t* src;
      bool ok;
      tile_of(i, src, ok);
      (void)src;
      const u32x4 z = {0u, 0u, 0u, 0u};
      lds[(buf * FRAGS + f) * 64 + lane] = (ok && ks < ks_e) ? r[i] : z;
    }
  };

  // ---- weight batches ----
  auto load_w = [&](int ks0, u32x4 (&wf)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int ks = ks0 + u;
      const int ksc = ks < ks_e ? ks : ks_e - 1;   // clamped: always a valid block; masked when used
      wf[u] = ONCE ? load_stream_16(wp + (size_t)ksc * W_KSTRIDE) : *reinterpret_cast<const u32x4*>(wp + (size_t)ksc * W_KSTRIDE);
    }
  };

  f32x16 acc[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[i][j] = 0.f;

  // One batch of U k-steps.  The activation fragments of k-step u + 1 are read from LDS while the matrix cores
  // work on k-step u (two register sets): with one wave per SIMD nothing else would hide the LDS latency.
  auto compute = [&](int buf, int kk0, int ks0, const u32x4 (&wf)[U]) {
    u32x4 xq[2][MT * PL];
    auto fetch = [&](int u, u32x4 (&dst)[MT * PL]) {
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int p = 0; p < PL; ++p) dst[m * PL + p] = lds[(buf * FRAGS + ((kk0 + u) * MT + m) * PL + p) * 64 + lane];
    };
    fetch(0, xq[0]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u + 1 < U) fetch(u + 1, xq[(u + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);          // the reads above are issued before the multiplies below
      const bool ok = ks0 + u < ks_e;             // uniform; past the end the weights count as zero
      const u32x4 z = {0u, 0u, 0u, 0u};
      const h16x8 w1 = ok ? wf[u] : z;
#pragma unroll
      for (int p = PL - 1; p >= 0; --p)           // small term first; the MT products of a term are independent
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[m] = mfma_32x32x16<FMT>(w1, xq[u & 1][m * PL + p], acc[m]);
    }
  };

  // Ring of R weight batches in registers: while batch b is multiplied, batches b+1 .. b+R-1 are in
  // flight.  A group of R batches spans R/NBC activation chunks; k-steps past the end are masked to zero.
  constexpr int R = 4;
  constexpr int NBC = KC / U;                       // batches per activation chunk (divides R)
  const int n_groups = (ks_e - ks_b + R * U - 1) / (R * U);
  u32x4 wr[R][U];
  u32x4 xr[PT];
  stage_load(0, xr);
#pragma unroll
  for (int r = 0; r < R - 1; ++r) load_w(ks_b + r * U, wr[r]);
  __builtin_amdgcn_sched_barrier(0);
  stage_store(0, xr);
  __syncthreads();
  // the factors are complete here (their loads are as old as the first chunk's); the empty statement keeps the
  // compiler from moving the fetch down to the epilogue, where it would cost a round trip at the end of the kernel
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    rs[m] = (a.x_ss && !grouped) ? row_rstd(a, ssq[m]) : 1.f;
    asm volatile("" : "+v"(rs[m]));
  }
  for (int g = 0; g < n_groups; ++g) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int b = g * R + r;
      const int c = g * (R / NBC) + r / NBC;
      if (r % NBC == 0) stage_load(c + 1, xr);
      load_w(ks_b + (b + R - 1) * U, wr[(r + R - 1) % R]);
      // keep the issue order: the loads above go out before the multiply below starts waiting
      __builtin_amdgcn_sched_barrier(0);
      compute(c & 1, (r % NBC) * U, ks_b + b * U, wr[r]);
      __builtin_amdgcn_sched_barrier(0);
      if (r % NBC == NBC - 1) {
        stage_store(c + 1, xr);
        __syncthreads();
      }
    }
  }
  if (!have_tile) return;
  if (PL != 2) fetch_lm_rows();
  if constexpr (EPI == EPI_LMHEAD)                   // past the last barrier: the activation chunks are dead
    lmhead_epilogue<1, MT, true>(a, reinterpret_cast<f32x4*>(lds) + wave * 4 * WAVE, reinterpret_cast<const f32x16(&)[1][MT]>(acc),
                           lm, nt, mt0, nt, n_tiles, lane);
  else
    tile_epilogue<MT, EPI, PL, FMT>(a, acc, nt, n_tiles, mt0, split, row_base, lane, rs);
}

// ---- expert-grouped decode form: up to 32 rows per expert, J tile groups per workgroup ----
// At decode an expert receives a handful of rows, and the skinny form above then spends a tenth of its time on
// the activations: every workgroup stages all K of the expert's rows for the 128 weight rows it owns, so the rows
// are fetched as often as the expert has tile groups, with gather loads that touch sixteen cache lines for eight
// useful rows (measured at the 30B-A3B shape: gate/up 154 us with the activation loads, 144 us without, 135 us for a
// kernel that only streams the same weights).  Here a workgroup takes J consecutive tile groups of one expert: wave w
// owns tile w of each of them, the activation chunk in LDS serves all J, and a workgroup lives J times as long, so
// that the routing look-up, the first chunk and the epilogue are paid a J-th as often.  With the interleaved weight
// layout the J groups are J contiguous runs of 4 KB per k-step.  Per accumulator the products come in the order of
// the skinny form (k ascending, small term first): the results are the same bits.
//
// A chunk is KC k-steps of activations in LDS; its weight batches are taken in the order (first half of the chunk:
// tile group 0 .. J-1, second half: 0 .. J-1), U = KC / 2 k-steps each, through a ring of R batches in registers.
// (Four groups per workgroup leave registers for 4 KB batches only, which was measured slower than one group.)
template <int J>
struct ExpertTiling {
  static constexpr int KC = 16, U = J == 1 ? 4 : 8, NBC = KC / U;
  static constexpr int BPC = J * NBC;                    // weight batches per chunk
  static constexpr int R = (BPC % 4 == 0) ? 4 : 3;       // ring depth: divides BPC, so ring slots are static
  static_assert(BPC % R == 0, "ring depth must divide the batches of a chunk");
};

template <int J, int EPI, int PL, int FMT>
__global__ __launch_bounds__(GEMM_THREADS) void gemm_expert_kernel(GemmArgs a) {
  using TL = ExpertTiling<J>;
  constexpr int KC = TL::KC, U = TL::U, BPC = TL::BPC, R = TL::R;
  constexpr int FRAGS = KC * PL, PT = FRAGS / GEMM_WAVES;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  u32x4* lds = reinterpret_cast<u32x4*>(lds_raw);   // [2][FRAGS][64 lanes]

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r32 = lane & 31, half = lane >> 5;
  const int mt0 = blockIdx.z;                       // 32-row tile of the expert's rows
  // REACHED (J == 1): only experts that have rows get workgroups.  blockIdx.x counts through those (the ids past them leave),
  // so that the live workgroups are the first ones and spread evenly over the units; otherwise blockIdx.y is the expert.
  constexpr bool REACHED = J == 1;
  int e = blockIdx.y, bx = blockIdx.x;
  int prev = -1;                                    // the expert with rows before e, or -1
  bool last = false;                                // e is the last one with rows
  unsigned long long has[4];                        // bit e % 64 of word e / 64: expert e has rows (uniform)
  auto pick = [&]() -> bool {                       // e, prev and last from the workgroup's place among the live ones; false: none
    const int rank = blockIdx.x / a.expert_wgs;
    bx = blockIdx.x % a.expert_wgs;
    e = -1;
    int n = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int rk = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(has[w] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)has[w], 0));
      const bool set = (has[w] >> lane) & 1ull;
      const unsigned long long at = __ballot(set && rk == rank), before = __ballot(set && rk == rank - 1);
      if (at) e = 64 * w + __builtin_ctzll(at);
      if (before) prev = 64 * w + __builtin_ctzll(before);
      n += __popcll(has[w]);
    }
    last = rank == n - 1;
    return e >= 0;
  };
  int row_base, my_pair = -1;
  if (a.route_idx) {
    // No grouping pass: the workgroup reads the routing table (a few KB, the same for every workgroup of the launch)
    // and finds what a counting sort by expert would have told it: how many pairs go to experts before this one
    // (row_base), how many to this one, and which, in pair order.  Thread i looks at the pairs i * PPT .. + PPT - 1,
    // so thread order is pair order.  One round trip, as the look-up of the sorted lists was.  The first workgroup
    // of each expert publishes the result (first row per expert, row of every pair) for the kernels that follow.
    __shared__ int32_t route_sum[GEMM_WAVES][2];
    __shared__ int32_t route_rows[32];              // pairs of this workgroup's tile of the expert's rows
    const int ppt = (a.n_pairs + GEMM_THREADS - 1) / GEMM_THREADS;
    const int p0 = (int)threadIdx.x * ppt;
    if constexpr (REACHED) {
      __shared__ uint8_t route_has[256];
      route_has[threadIdx.x] = 0;
      __syncthreads();
      for (int i = 0; i < ppt; ++i) {
        const int idx = p0 + i < a.n_pairs ? a.route_idx[p0 + i] : -1;
        if (idx >= 0 && idx < 256) route_has[idx] = 1;
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < 4; ++w) has[w] = __ballot(route_has[64 * w + lane] != 0);
      if (!pick()) {                                // uniform over the workgroup
        // no expert has rows: the table that the next kernels index with is still published, all empty
        if (!(has[0] | has[1] | has[2] | has[3]) && blockIdx.x == 0 && mt0 == 0)
          for (int i = threadIdx.x; i <= a.n_experts; i += GEMM_THREADS) a.pub_group_off[i] = 0;
        return;
      }
    }
    int less = 0, eq = 0;
    for (int i = 0; i < ppt; ++i) {
      const int p = p0 + i;
      const int idx = p < a.n_pairs ? a.route_idx[p] : 0x7FFFFFFF;
      less += idx < e ? 1 : 0;
      eq += idx == e ? 1 : 0;
    }
    int incl = eq;                                  // inclusive prefix of the matches over the wave's lanes
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o, WAVE);
      if (lane >= o) incl += v;
    }
    less = (int)wave_sum((float)less);              // at most 4096 pairs: exact in fp32
    if (lane == 63) { route_sum[wave][0] = less; route_sum[wave][1] = incl; }
    if (threadIdx.x < 32) route_rows[threadIdx.x] = -1;
    __syncthreads();
    row_base = 0;
    int n_rows = 0, before = 0;
#pragma unroll
    for (int w = 0; w < GEMM_WAVES; ++w) {
      row_base += route_sum[w][0];
      if (w < wave) before += route_sum[w][1];
      n_rows += route_sum[w][1];
    }
    a.T = n_rows;
    if constexpr (REACHED) {
      if (bx == 0 && mt0 == 0) {                    // its own first row, that of the experts without rows before it ...
        for (int i = prev + 1 + (int)threadIdx.x; i <= e; i += GEMM_THREADS) a.pub_group_off[i] = row_base;
        if (last)                                   // ... and of those behind the last one
          for (int i = e + 1 + (int)threadIdx.x; i <= a.n_experts; i += GEMM_THREADS) a.pub_group_off[i] = row_base + n_rows;
      }
    } else if (bx == 0 && mt0 == 0 && threadIdx.x == 0) {   // also for an expert without rows
      a.pub_group_off[e] = row_base;
      if (e == (int)gridDim.y - 1) a.pub_group_off[e + 1] = row_base + n_rows;
    }
    if (mt0 * 32 >= a.T) return;                    // uniform over the workgroup
    int pos = before + incl - eq - mt0 * 32;        // place, inside this tile, of the thread's first match
    for (int i = 0; i < ppt; ++i) {
      const int p = p0 + i;
      if (p < a.n_pairs && a.route_idx[p] == e) {   // another look at the same few entries: cache hits
        if (pos >= 0 && pos < 32) route_rows[pos] = p;
        ++pos;
      }
    }
    __syncthreads();
    my_pair = route_rows[r32];                      // -1 past the expert's last row
    if (bx == 0) {
      if (threadIdx.x < 32 && my_pair >= 0) a.pub_pair_pos[my_pair] = row_base + mt0 * 32 + r32;
    }
  } else {
    if constexpr (REACHED) {
      int first[4], next[4];                        // all on their way before the first is used
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        first[w] = a.group_off[min(64 * w + lane, a.n_experts)];
        next[w] = a.group_off[min(64 * w + lane + 1, a.n_experts)];
      }
#pragma unroll
      for (int w = 0; w < 4; ++w) has[w] = __ballot(next[w] > first[w]);
      if (!pick()) return;                          // uniform over the workgroup, before any barrier
    }
    row_base = a.group_off[e];
    a.T = a.group_off[e + 1] - row_base;
    if (mt0 * 32 >= a.T) return;                    // uniform over the workgroup, before any barrier
  }
  const h16_t* wbase = a.w[0] + (size_t)e * a.w_expert_stride;

  const int KS = a.K >> 4;
  const int n_tiles = (a.N + 31) >> 5;
  // tile of this wave in tile group j: (bx * J + j) * 4 + wave; consecutive groups lie KS * W_KSTRIDE apart
  const int nt0 = bx * J * W_GROUP + wave;
  static_assert(W_GROUP == GEMM_WAVES, "a wave owns one tile of every interleaved group");
  const h16_t* wp = wbase + packed_tile_offset(nt0, KS) + lane * 8;
  const size_t group_stride = (size_t)KS * W_KSTRIDE;
  // a tile group past the end of the matrix is read as the last one that exists (cache hits) and never stored
  int jmax = ((n_tiles + W_GROUP - 1) / W_GROUP) - 1 - bx * J;
  if (jmax > J - 1) jmax = J - 1;

  // ---- activation staging: each wave moves PT fragments of a chunk; fragment f = (k-step f / PL, plane f % PL) ----
  const int r = mt0 * 32 + r32;
  const bool xok = r < a.T;
  const h16_t* xsrc;
  float rs[1];
  f32x4 ssq;
  {
    const int rr = xok ? r : 0;
    int row;
    if (a.route_idx) row = my_pair >= 0 ? my_pair / a.top_k : 0;       // the pair's token
    else row = a.x_rows ? a.x_rows[row_base + rr] : row_base + rr;
    xsrc = a.x + frag_act_offset(row, 8 * half, 0, a.x_mtiles, PL);
    ssq = f32x4{1.f, 1.f, 1.f, 1.f};
    if (a.x_ss && a.route_idx) ssq = row_ss(a, row);              // the pair's token is the activation row
    __builtin_amdgcn_sched_barrier(0);
  }
  const size_t x_kstride = (size_t)a.x_mtiles * PL * 512;
  auto stage_load = [&](int chunk, u32x4 (&rg)[PT]) {
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int f = wave + GEMM_WAVES * i;
      const int ks = chunk * KC + f / PL, p = f % PL;
      const int ksc = ks < KS ? ks : KS - 1;         // clamped: always a valid fragment; masked when stored
      rg[i] = *reinterpret_cast<const u32x4*>(xsrc + (size_t)ksc * x_kstride + (size_t)p * 512);
    }
  };
  auto stage_store = [&](int chunk, const u32x4 (&rg)[PT]) {
    const int buf = chunk & 1;
    const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int f = wave + GEMM_WAVES * i;
      const int ks = chunk * KC + f / PL;
      lds[(buf * FRAGS + f) * 64 + lane] = (xok && ks < KS) ? rg[i] : z;
    }
  };

  // ---- weight batches: batch s of chunk c = tile group s % J, k-steps c * KC + (s / J) * U .. + U ----
  auto load_w = [&](int c, int s, u32x4 (&wf)[U]) {
    const int j = s % J;
    const h16_t* base = wp + (size_t)(j < jmax ? j : jmax) * group_stride;
    const int ks0 = c * KC + (s / J) * U;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int ks = ks0 + u;
      const int ksc = ks < KS ? ks : KS - 1;         // clamped: always a valid block; masked when used
      wf[u] = load_stream_16(base + (size_t)ksc * W_KSTRIDE);
    }
  };

  f32x16 acc[J];
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[j][q] = 0.f;

  auto compute = [&](int buf, int kk0, int ks0, const u32x4 (&wf)[U], f32x16& ac) {
    u32x4 xq[2][PL];
    auto fetch = [&](int u, u32x4 (&dst)[PL]) {
#pragma unroll
      for (int p = 0; p < PL; ++p) dst[p] = lds[(buf * FRAGS + (kk0 + u) * PL + p) * 64 + lane];
    };
    fetch(0, xq[0]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u + 1 < U) fetch(u + 1, xq[(u + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);          // the reads above are issued before the multiplies below
      const bool ok = ks0 + u < KS;               // uniform; past the end the weights count as zero
      const u32x4 z = {0u, 0u, 0u, 0u};
      const h16x8 w1 = ok ? wf[u] : z;
#pragma unroll
      for (int p = PL - 1; p >= 0; --p) ac = mfma_32x32x16<FMT>(w1, xq[u & 1][p], ac);   // small term first
    }
  };

  const int n_chunks = (KS + KC - 1) / KC;
  u32x4 wr[R][U];
  u32x4 xr[PT];
  stage_load(0, xr);
  __builtin_amdgcn_sched_barrier(0);                // the activation loads are older than every weight load
#pragma unroll
  for (int s = 0; s < R - 1; ++s) load_w(0, s, wr[s]);
  __builtin_amdgcn_sched_barrier(0);
  stage_store(0, xr);
  __syncthreads();
  rs[0] = (a.x_ss && a.route_idx) ? row_rstd(a, ssq) : 1.f;   // as in the skinny form: fetched first, finished here
  asm volatile("" : "+v"(rs[0]));
  for (int c = 0; c < n_chunks; ++c) {
    stage_load(c + 1, xr);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < BPC; ++s) {
      // batch s + R - 1 of this chunk, or the first batches of the next one, goes out before batch s is multiplied
      const int sn = s + R - 1;
      if (sn < BPC) load_w(c, sn, wr[sn % R]); else load_w(c + 1, sn - BPC, wr[sn % R]);
      __builtin_amdgcn_sched_barrier(0);
      compute(c & 1, (s / J) * U, c * KC + (s / J) * U, wr[s % R], acc[s % J]);
      __builtin_amdgcn_sched_barrier(0);
    }
    stage_store(c + 1, xr);
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int nt = nt0 + j * W_GROUP;
    if (nt < n_tiles)
      tile_epilogue<1, EPI, PL, FMT>(a, reinterpret_cast<const f32x16(&)[1]>(acc[j]), nt, n_tiles, mt0, 0, row_base, lane, rs);
  }
}

std::atomic<int> g_units{256};                       // compute units of the device (gemm_set_units): every model on it sets the same value

template <int MT, int EPI, int PL, int FMT, bool ONCE>
void launch_one_form(const GemmArgs& a, dim3 grid, hipStream_t st) {
  static std::once_flag attr_once;                  // raise the dynamic LDS limit once per instantiation, from any thread
  constexpr int lds = Tiling<MT, PL>::LDS_BYTES;
  std::call_once(attr_once, [] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_skinny_kernel<MT, EPI, PL, FMT, ONCE>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  });
  hipLaunchKernelGGL((gemm_skinny_kernel<MT, EPI, PL, FMT, ONCE>), grid, dim3(GEMM_THREADS), lds, st, a);
}

// Several token tiles (grid z) share a weight tile only in the store form at 64 tokens per tile (two-group calls) and
// in the 128-token forms, of which SwiGLU on two terms has no more than one (longer dense calls take the long-call form);
// an expert group with more rows than a tile is rare enough to keep the streaming mark.
template <int MT, int EPI, int PL, int FMT>
void launch_one(const GemmArgs& a, dim3 grid, hipStream_t st) {
  constexpr bool shared_tiles_possible = (MT == 4 && !(EPI == EPI_SWIGLU && PL == 2)) || (MT == 2 && EPI == EPI_STORE);
  if (shared_tiles_possible && grid.z > 1 && a.group_off == nullptr) launch_one_form<MT, EPI, PL, FMT, !shared_tiles_possible>(a, grid, st);
  else launch_one_form<MT, EPI, PL, FMT, true>(a, grid, st);
}

// formats built: bf16 activations as one or two terms, fp16 activations as one term; LM heads of more than 64 rows on two
// terms take the long-call form (gemm_lmhead refuses them)
template <int MT, int EPI>
void launch_fmt(const GemmArgs& a, dim3 grid, const Act& x, hipStream_t st) {
  if (x.dtype == DT_F16) {
    launch_one<MT, EPI, 1, DT_F16>(a, grid, st);
  } else if (x.planes == 2) {
    if constexpr (!(MT == 4 && EPI == EPI_LMHEAD)) launch_one<MT, EPI, 2, DT_BF16>(a, grid, st);
  } else {
    launch_one<MT, EPI, 1, DT_BF16>(a, grid, st);
  }
}

template <int EPI>
void launch_mt(const GemmArgs& a, int n_tiles, int grid_y, int mt, const Act& x, hipStream_t st) {
  const int gx = (n_tiles + GEMM_WAVES - 1) / GEMM_WAVES;
  const int mtiles = (a.T + 31) / 32;
  if (mt == 1) launch_fmt<1, EPI>(a, dim3(gx, grid_y, mtiles), x, st);
  else if (mt == 2) launch_fmt<2, EPI>(a, dim3(gx, grid_y, (mtiles + 1) / 2), x, st);
  else launch_fmt<4, EPI>(a, dim3(gx, grid_y, (mtiles + 3) / 4), x, st);
}

// Expert-grouped decode form (two-term bf16 only; the other formats keep the skinny form).  Tile groups per workgroup:
//  - One, for the experts that have rows, where a batch reaches few of them.  With a workgroup of three groups for every
//    expert the empty ones, resident for as long as it takes to find out, left some units two full ones and others
//    none, and a batch of one put its eight experts on 32 units (30B-A3B shape, us of gate/up + down, before -> now: 1 token
//    72 -> 31, 4 tokens 100 -> 62, 12 131 -> 114, 16 144 -> 131, 24 161 -> 160; 32 tokens, 88 % of the experts: 173, 178).
//  - Otherwise three or two, whichever divides the groups of an expert and still leaves two workgroups per compute
//    unit (measured at the 30B-A3B shape: gate/up, 12 groups, 155 us with one group per workgroup, 145 with two, 146
//    with three; down, 16 groups, 77.7 / 77.0 / 78.8); a grid that cannot fill the device anyway takes two.
template <int J, int EPI>
void launch_expert_one(const GemmArgs& a, dim3 grid, hipStream_t st) {
  static std::once_flag attr_once;
  constexpr int lds = 2 * ExpertTiling<J>::KC * 2 * 1024;
  std::call_once(attr_once, [] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_expert_kernel<J, EPI, 2, DT_BF16>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  });
  hipLaunchKernelGGL((gemm_expert_kernel<J, EPI, 2, DT_BF16>), grid, dim3(GEMM_THREADS), lds, st, a);
}

int expert_tile_groups(int n_tiles, int n_experts, int n_pairs, int n_units) {
  const int groups = (n_tiles + W_GROUP - 1) / W_GROUP;
  // share of the experts that a random routing of so many pairs misses
  if (groups == 1 || powf(1.f - 1.f / (float)n_experts, (float)n_pairs) > 0.2f) return 1;
  for (int j = 3; j >= 2; --j)
    if (groups % j == 0 && (long)(groups / j) * n_experts >= 2L * n_units) return j;
  return 2;
}

template <int EPI>
bool launch_expert(GemmArgs a, int n_tiles, int n_experts, int n_pairs, const Act& x, hipStream_t st) {
  if (x.planes != 2 || x.dtype != DT_BF16) return false;
  const int j = expert_tile_groups(n_tiles, n_experts, n_pairs, g_units.load(std::memory_order_relaxed));
  const int groups = (n_tiles + W_GROUP - 1) / W_GROUP, row_tiles = (a.T + 31) / 32;
  a.n_experts = n_experts; a.expert_wgs = (groups + j - 1) / j;
  if (j == 1) launch_expert_one<1, EPI>(a, dim3(a.expert_wgs * (n_pairs < n_experts ? n_pairs : n_experts), 1, row_tiles), st);
  else if (j == 2) launch_expert_one<2, EPI>(a, dim3(a.expert_wgs, n_experts, row_tiles), st);
  else launch_expert_one<3, EPI>(a, dim3(a.expert_wgs, n_experts, row_tiles), st);
  return true;
}

// token tiles per workgroup
int pick_mt(int T) { return T <= 32 ? 1 : (T <= 64 ? 2 : 4); }

void fill_x(GemmArgs& a, const Act& x) {
  a.x = x.p; a.x_mtiles = x.mtiles();
  a.x_ss = x.ss; a.x_eps = x.eps;
}

}  // namespace

// Store GEMMs of 65..128 tokens run as two 64-token groups (the weights of these small matrices are read twice,
// the second time from cache): measured faster than one 128-token tile (MoE decode q|k|v 1.03 -> 0.75 ms per step,
// output projection 0.91 -> 0.66, router 0.56 -> 0.44 with the split planning that knows of the two groups; the same
// trick one size down, two 32-token groups for 33..64 tokens, was measured slower).
static int store_mt(int T) { return (T > 64 && T <= 128) ? 2 : pick_mt(T); }
static int store_token_groups(int T) { return (T > 64 && T <= 128) ? 2 : 1; }

int gemm_max_splits() { return 16; }

void gemm_set_units(int n_units) { g_units.store(n_units > 0 ? n_units : 1, std::memory_order_relaxed); }

// Split-K planning.  A compute unit takes in only so many bytes per microsecond however many waves it holds, so
// what counts is that every unit gets the same number of bytes: the grid is kept at or just under one workgroup
// per unit (a grid of 1.2 workgroups per unit takes as long as one of 2), with as few planes as that allows.
static int ksteps_for(int K, int splits) { return (K / 16 + splits - 1) / splits; }

// k-steps that one round of the skinny form's main loop covers (a ring of four weight batches); a K range that is
// not a multiple of it is padded with masked k-steps whose loads are still issued
static int kstep_round(int T, int planes, int dtype) {
  const int mt = store_mt(T);
  const int pl = dtype == DT_F16 ? 1 : planes;
  const int kc = (mt == 1 && pl == 2) ? 12 : ((32 / (mt * pl)) > 16 ? 16 : (32 / (mt * pl)));   // Tiling<MT, PL>::KC
  return 2 * kc;
}

int gemm_plan_splits(int N, int K, int T, int max_splits, int n_units, int planes, int dtype) {
  const int per = GEMM_WAVES;                                          // weight tiles per workgroup
  const int groups = ((N + 31) / 32 + per - 1) / per * store_token_groups(T);   // workgroups per split
  const int KS = K / 16;
  int want = n_units / groups;                      // floor: never more workgroups than units
  if (want > max_splits) want = max_splits;
  if (want > KS / 8) want = KS / 8;                 // at least eight k-steps per split
  if (want < 1) want = 1;
  // A workgroup's time goes with the k-steps its loop runs, padding included, so among the split counts that fit the
  // device the one with the fewest padded k-steps per split wins, and of several such the one with the fewest planes
  // (measured at the 4B shape, 64 tokens: output projection, K = 4096, 12 planes 11.2 us, 8 planes 9.9 us; down
  // projection, K = 9728, 12 planes 17.4 us, 10 planes 16.4 us: both pad 22 and 51 k-steps to 32 and 64).
  const int round = kstep_round(T, planes, dtype);
  int best = 1, best_padded = 0x7FFFFFFF;
  for (int s = 1; s <= want; ++s) {
    const int ksper = ksteps_for(K, s);
    const int padded = (ksper + round - 1) / round * round;
    if (padded < best_padded) { best_padded = padded; best = s; }
  }
  const int ksper = ksteps_for(K, best);
  return (KS + ksper - 1) / ksper;                  // no empty split
}

hipError_t gemm_store(const LinearW& w, const Act& x, int T, float* y, int ldy, int splits, hipStream_t st) {
  GemmArgs a = {};
  fill_x(a, x);
  int tiles = 0;
  for (int i = 0; i < 3; ++i) { a.w[i] = w.seg[i]; a.w_tiles[i] = (w.rows[i] + 31) / 32; tiles += a.w_tiles[i]; }
  a.N = w.N; a.K = w.K; a.T = T;
  a.ksteps_per_split = ksteps_for(w.K, splits);   // same rule as gemm_plan_splits
  a.y = y; a.ldy = ldy;
  launch_mt<EPI_STORE>(a, tiles, splits, store_mt(T), x, st);
  return hipGetLastError();
}

hipError_t gemm_swiglu(const h16_t* w_gate_up, int F, int K, const Act& x, int T, const Act& act, hipStream_t st) {
  GemmArgs a = {};
  fill_x(a, x);
  a.w[0] = w_gate_up; a.w_tiles[0] = F / 16;
  a.N = 2 * F; a.K = K; a.T = T;
  a.ksteps_per_split = K / 16;
  a.act = act.p; a.act_mtiles = act.mtiles();
  launch_mt<EPI_SWIGLU>(a, a.w_tiles[0], 1, pick_mt(T), x, st);
  return hipGetLastError();
}

// Token-tile height of the expert-grouped kernels.  An expert's weights are streamed once per tile of 32 * mt rows
// and every tile reads 32 * mt activation rows whether or not they exist, so the tile should just cover the rows an
// expert is expected to get (decode: a handful; prefill: hundreds); the grid covers max_rows and workgroups past an
// expert's last row exit at once.
static int grouped_mt(int expected_rows) {
  return expected_rows <= 16 ? 1 : (expected_rows <= 40 ? 2 : 4);
}

static int rows_expected(int n_pairs, int E) { return (n_pairs + E - 1) / E; }

hipError_t gemm_grouped_swiglu(const h16_t* w_gate_up, int E, int F, int K, const Act& x, const int32_t* x_rows,
                               const int32_t* group_off, int max_rows, int n_pairs, const Act& act,
                               hipStream_t st) {
  if (x.ss && x_rows) return hipErrorInvalidValue;   // the epilogue would need the row list to find a row's factor
  GemmArgs a = {};
  fill_x(a, x);
  a.x_rows = x_rows;
  a.w[0] = w_gate_up; a.w_tiles[0] = F / 16;
  a.N = 2 * F; a.K = K; a.T = max_rows;
  a.ksteps_per_split = K / 16;
  a.act = act.p; a.act_mtiles = act.mtiles();
  a.group_off = group_off; a.w_expert_stride = packed_weight_elems(2 * F, K);
  if (grouped_mt(rows_expected(n_pairs, E)) == 1 && launch_expert<EPI_SWIGLU>(a, a.w_tiles[0], E, n_pairs, x, st)) return hipGetLastError();
  launch_mt<EPI_SWIGLU>(a, a.w_tiles[0], E, grouped_mt(rows_expected(n_pairs, E)), x, st);
  return hipGetLastError();
}

hipError_t gemm_grouped_store(const h16_t* w, int E, int N, int K, const Act& x, const int32_t* group_off,
                              int max_rows, int n_pairs, float* y, hipStream_t st) {
  GemmArgs a = {};
  fill_x(a, x);
  a.w[0] = w; a.w_tiles[0] = (N + 31) / 32;
  a.N = N; a.K = K; a.T = max_rows;
  a.ksteps_per_split = K / 16;
  a.y = y; a.ldy = N;
  a.group_off = group_off; a.w_expert_stride = packed_weight_elems(N, K);
  if (grouped_mt(rows_expected(n_pairs, E)) == 1 && launch_expert<EPI_STORE>(a, a.w_tiles[0], E, n_pairs, x, st)) return hipGetLastError();
  launch_mt<EPI_STORE>(a, a.w_tiles[0], E, grouped_mt(rows_expected(n_pairs, E)), x, st);
  return hipGetLastError();
}

// Routed form of the expert-grouped gate/up GEMM at decode: no grouping pass; every workgroup finds its expert's
// pairs in the routing table (route_idx[token * top_k + slot] = expert), reads the token's row of x and writes act
// in expert order (pairs of expert 0 first, in pair order: what the counting sort produces).  The launch also
// publishes group_off[E + 1] and pair_pos[n_pairs] of that order, which the down GEMM and the combine then read.
bool gemm_routed_form(int E, const Act& x, int n_pairs) {
  if (x.planes != 2 || x.dtype != DT_BF16 || grouped_mt(rows_expected(n_pairs, E)) != 1) return false;
  return n_pairs <= 16 * GEMM_THREADS;              // at most 16 table entries per thread of a workgroup
}

hipError_t gemm_routed_swiglu(const h16_t* w_gate_up, int E, int F, int K, const Act& x, const int32_t* route_idx,
                              int n_pairs, int top_k, int max_rows, const Act& act, int32_t* group_off,
                              int32_t* pair_pos, hipStream_t st) {
  GemmArgs a = {};
  fill_x(a, x);
  a.w[0] = w_gate_up; a.w_tiles[0] = F / 16;
  a.N = 2 * F; a.K = K; a.T = max_rows;
  a.ksteps_per_split = K / 16;
  a.act = act.p; a.act_mtiles = act.mtiles();
  a.w_expert_stride = packed_weight_elems(2 * F, K);
  a.route_idx = route_idx; a.n_pairs = n_pairs; a.top_k = top_k;
  a.pub_group_off = group_off; a.pub_pair_pos = pair_pos;
  if (!launch_expert<EPI_SWIGLU>(a, a.w_tiles[0], E, n_pairs, x, st)) return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t gemm_lmhead(const h16_t* w_lm, int V, int K, const Act& x, int T, float* logits, float* part,
                       const uint64_t* seeds, const float* temperature, const int32_t* sample_pos,
                       const int32_t* row_seq, bool draw, hipStream_t st) {
  if (x.ss) return hipErrorInvalidValue;              // the LM-head epilogue takes finished rows only
  if (x.planes == 2 && pick_mt(T) == 4) return hipErrorInvalidValue;
  GemmArgs a = {};
  fill_x(a, x);
  a.w[0] = w_lm; a.w_tiles[0] = (V + 31) / 32;
  a.N = V; a.K = K; a.T = T;
  a.ksteps_per_split = K / 16;
  a.logits = logits; a.part = part; a.seeds = seeds; a.temperature = temperature; a.sample_pos = sample_pos;
  a.row_seq = row_seq; a.draw = draw ? 1 : 0;
  launch_mt<EPI_LMHEAD>(a, a.w_tiles[0], 1, pick_mt(T), x, st);
  return hipGetLastError();
}

}  // namespace rlx
