// GEMM of long calls (prefill and scoring chunks, LM heads of many rows) on two-term bf16 activations.
//
//   y[t, n] = sum_k x[t, k] * W[n, k],  x = hi + lo: two MFMA 32x32x16 per weight fragment and 32 x 32 outputs
//
// A workgroup of WR x WT waves computes 32 JW WR weight rows x 32 MW WT tokens, a wave 32 JW x 32 MW of them (JW weight tiles x
// MW token tiles: 16 JW MW accumulator registers).  Both operands pass through LDS, copied there by the hardware
// (global_load_lds, 16 bytes per lane, no registers in between), in stages of 32 k, NB stage buffers deep.
//  - Weights: the packed layout's fragments, 1 KB per copy, read back linearly.
//  - Activations: rows (Act::pitch): the 32 k of a stage are one 128-byte line of a row (eight 16-byte chunks: per
//    8 k the large terms, then the small ones), so any list of rows can be gathered a full line at a time; a copy
//    takes eight rows.  In LDS row r's chunk c sits in slot c ^ ((r >> 1) & 7) of the row's 128 bytes (the copy picks
//    the chunk per lane), which spreads the 16 rows that a fragment read touches at a time over all 64 banks.
// What bounds it: the matrix cores under the card's power limit (the same loop without copies and LDS reads runs at
// 1.57-1.67 PFLOP/s on random data and at 2.07 on zeros) and the copies: issued in a burst after the barrier they
// hold up the waves' own products, so they are spread over the stage, two per eight products.  Measured at 32 768
// tokens, K 2560, N 6144: 1.24 PFLOP/s (both terms counted) with the burst, 1.31 spread; stores of 16 bytes per lane
// to 32 rows at a time 1.33, of 128-byte lines (the store form swaps the operands, so that lanes run along n) 1.36.
// Per accumulator the products come in the order of the skinny form (k ascending, small term first).
#include <mutex>

#include "gemm_core.h"
#include "lds_copy.h"

namespace rlx {
namespace {

template <int JW, int MW, int WR, int WT, int NB>
struct LongTiling {
  static constexpr int WAVES = WR * WT, ROWS = 32 * JW * WR, TOKENS = 32 * MW * WT;
  static constexpr int WFR = 2 * JW * WR, XFR = 4 * MW * WT;       // KB of weights and of activations per stage
  static constexpr int STAGE = (WFR + XFR) * 1024;
  static constexpr int PW = (WFR + WAVES - 1) / WAVES, PX = XFR / WAVES, P = PW + PX;   // copies per wave and stage
  static constexpr int LM_TILES = JW % 2 ? JW : 2;                 // weight tiles of an LM head's part
  static constexpr int LDS_BYTES = NB * STAGE, LM_SCRATCH = WAVES * LM_TILES * 4096;
  static_assert(XFR % WAVES == 0, "the waves share a stage's activations evenly");
};

// grid: 8 * ceil(tiles / 8) workgroups, tiles = splits x weight tiles x (token tiles, or items of the list).  The ids go
// round robin over the eight XCDs, so XCD x takes every eighth id; each takes one contiguous eighth of the tiles, whose
// order keeps the tiles in flight on an XCD close: `band` token tiles, then the next weight tile.
template <int JW, int MW, int WR, int WT, int NB, int EPI>
__global__ __launch_bounds__(64 * WR * WT) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_long_kernel(GemmArgs a, int n_wt,
                                                                                                           int n_tt, int band) {
  using TL = LongTiling<JW, MW, WR, WT, NB>;
  constexpr int NW = TL::WAVES, STAGE = TL::STAGE, PW = TL::PW, PX = TL::PX, P = TL::P, WFR = TL::WFR;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r32 = lane & 31, half = lane >> 5;
  const int wr = wave % WR, wt = wave / WR;

  // ---- the workgroup's tile ----
  if (a.item_expert) { n_tt = min(a.n_items[0], n_tt); band = 1; }
  const int per_split = n_wt * n_tt, tiles = per_split * a.splits;
  int id;
  {
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int base = tiles >> 3, extra = tiles & 7;
    if (j >= base + (xcd < extra ? 1 : 0)) return;   // uniform over the workgroup, before any barrier
    id = xcd * base + min(xcd, extra) + j;
  }
  const int split = id / per_split;
  id -= split * per_split;
  const int b0 = id / (band * n_wt) * band, h = min(band, n_tt - b0), in_band = id - b0 * n_wt;
  const int tw = in_band / h;
  int tt = b0 + in_band % h;
  int row_base = 0;
  if (a.item_expert) {
    const int e = a.item_expert[tt];
    tt = a.item_tile[tt];
    row_base = a.group_off[e];
    a.T = a.group_off[e + 1] - row_base;
    a.w[0] += (size_t)e * a.w_expert_stride;
  }

  // ---- copies: wave w takes copies w, w + NW, ... of a stage's weights (k-step, tile) and activations (eight rows) ----
  const int KS = a.K >> 4;
  const int n_tiles = (a.N + 31) >> 5;
  const int ks_b = split * a.ksteps_per_split;       // even: the host cuts K between stages
  const int ks_e = min(ks_b + a.ksteps_per_split, KS);
  const int n_st = (ks_e - ks_b) >> 1;               // whole stages; an odd last k-step is half a stage more
  const int n_cp = (ks_e - ks_b + 1) >> 1;           // stages to copy
  const uint32_t lds0 = lds_address(lds_raw);
  const h16_t* wp[PW];
  // a wave short of a copy repeats the last one's bytes
  auto weight_copy = [&](int i) { return WFR % NW == 0 ? wave + NW * i : min(wave + NW * i, WFR - 1); };
  int wstep[PW];
#pragma unroll
  for (int i = 0; i < PW; ++i) {
    const int f = weight_copy(i), j = f % (JW * WR);
    int lt = tw * JW * WR + j;
    wstep[i] = 1;
    if (lt >= n_tiles) { lt = 0; wstep[i] = 0; }     // no such tile: one cached block, its products are never stored
    const h16_t* base = a.w[0];
    if (lt >= a.w_tiles[0]) {
      lt -= a.w_tiles[0];
      base = a.w[1];
      if (lt >= a.w_tiles[1]) { lt -= a.w_tiles[1]; base = a.w[2]; }
    }
    wp[i] = base + packed_tile_offset(lt, KS) + lane * 8;
  }
  // a token row past the end reads the group's first row: a row only reaches its own outputs, which are not stored
  const h16_t* xp[PX];
#pragma unroll
  for (int i = 0; i < PX; ++i) {
    const int r = 8 * (wave + NW * i) + (lane >> 3);
    int t = tt * TL::TOKENS + r;
    if (t >= a.T) t = 0;
    const int row = a.x_rows ? a.x_rows[row_base + t] : row_base + t;
    xp[i] = a.x + (size_t)row * a.x_pitch + (size_t)ks_b * 32 + (size_t)(((lane & 7) ^ ((r >> 1) & 7)) * 8);
  }
  auto copy_one = [&](int i, int s, int buf) {       // stages past the end repeat the last one: counts stay the same
    const int sc = min(s, n_cp - 1);
    const uint32_t dst = lds0 + buf * STAGE;
    if (i < PW) {
      const int f = weight_copy(i);
      const int ks = min(ks_b + 2 * sc + f / (JW * WR), KS - 1);   // the missing half of an odd last stage: any block
      copy_to_lds(wp[i] + (size_t)(ks * wstep[i]) * W_KSTRIDE, dst + f * 1024);
    } else {
      copy_to_lds(xp[i - PW] + (size_t)sc * 64, dst + (WFR + wave + NW * (i - PW)) * 1024);
    }
  };

  f32x16 acc[JW][MW];
#pragma unroll
  for (int j = 0; j < JW; ++j)
#pragma unroll
    for (int m = 0; m < MW; ++m)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[j][m][q] = 0.f;

  // ---- fragments from LDS ----
  const unsigned char* w_rd = lds_raw + JW * wr * 1024 + lane * 16;
  const unsigned char* x_rd[4];                      // by (k-step, term) of the stage
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int chunk = ((c >> 1) * 2 + half) * 2 + (c & 1);
    x_rd[c] = lds_raw + WFR * 1024 + (wt * 32 * MW + r32) * 128 + ((chunk ^ ((r32 >> 1) & 7)) * 16);
  }
  auto read_w = [&](int buf, int kk, h16x8 (&w)[JW]) {
#pragma unroll
    for (int j = 0; j < JW; ++j) w[j] = *reinterpret_cast<const u32x4*>(w_rd + buf * STAGE + (kk * JW * WR + j) * 1024);
  };
  auto read_x = [&](int buf, int kk, int p, h16x8 (&x)[MW]) {
#pragma unroll
    for (int m = 0; m < MW; ++m) x[m] = *reinterpret_cast<const u32x4*>(x_rd[kk * 2 + p] + buf * STAGE + m * 4096);
  };
  // half a phase: the store form swaps the operands, so that lanes run along n and registers along the tokens
  auto products = [&](const h16x8 (&w)[JW], const h16x8 (&x)[MW], int hf) {
#pragma unroll
    for (int j = JW * hf / 2; j < JW * (hf + 1) / 2; ++j)
#pragma unroll
      for (int m = 0; m < MW; ++m)
        acc[j][m] = EPI == EPI_STORE ? mfma_32x32x16<DT_BF16>(x[m], w[j], acc[j][m]) : mfma_32x32x16<DT_BF16>(w[j], x[m], acc[j][m]);
  };
  // copies of slot k (0..5): those of the stage NB - 1 ahead, into the buffer that the last barrier released
  constexpr int AHEAD = NB - 1;
  auto slot = [&](int k, int s, int fbuf) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < P; ++i)
      if (i * 6 / P == k) copy_one(i, s + AHEAD, fbuf);
    __builtin_amdgcn_sched_barrier(0);
  };

#pragma unroll
  for (int s = 0; s < AHEAD; ++s)
#pragma unroll
    for (int i = 0; i < P; ++i) copy_one(i, s, s);
  wait_copies_and_barrier<(AHEAD - 1) * P>();
  const int tok0 = tt * TL::TOKENS + wt * 32 * MW;        // the wave's first token (of its group)
  int buf = 0, fbuf = AHEAD;
  if (tok0 >= a.T) {
    // all of the wave's tokens lie past the last row: it only copies, and leaves its SIMD to the waves beside it
    for (int s = 0; s < n_st; ++s) {
#pragma unroll
      for (int i = 0; i < P; ++i) copy_one(i, s + AHEAD, fbuf);
      wait_copies_and_barrier<(AHEAD - 1) * P>();
      fbuf = fbuf + 1 == NB ? 0 : fbuf + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    return;
  }
  h16x8 w0[JW], w1[JW], xa[MW], xb[MW];
  read_w(0, 0, w0);
  read_x(0, 0, 1, xa);
  __builtin_amdgcn_sched_barrier(0);
  for (int s = 0; s < n_st; ++s) {
    const int nbuf = buf + 1 == NB ? 0 : buf + 1;
    read_x(buf, 0, 0, xb);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    products(w0, xa, 0);                             // k-step 0, small term
    slot(0, s, fbuf);
    products(w0, xa, 1);
    slot(1, s, fbuf);
    read_w(buf, 1, w1);
    read_x(buf, 1, 1, xa);
    __builtin_amdgcn_sched_barrier(0);
    products(w0, xb, 0);                             // k-step 0, large term
    slot(2, s, fbuf);
    products(w0, xb, 1);
    slot(3, s, fbuf);
    read_x(buf, 1, 0, xb);
    __builtin_amdgcn_sched_barrier(0);
    products(w1, xa, 0);                             // k-step 1, small term
    slot(4, s, fbuf);
    products(w1, xa, 1);
    slot(5, s, fbuf);
    __builtin_amdgcn_s_setprio(0);
    wait_copies_and_barrier<(AHEAD - 1) * P>();      // stage s + 1 is in LDS; nobody reads stage s from here on
    read_w(nbuf, 0, w0);
    read_x(nbuf, 0, 1, xa);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    products(w1, xb, 0);                             // k-step 1, large term
    products(w1, xb, 1);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
    buf = nbuf;
    fbuf = fbuf + 1 == NB ? 0 : fbuf + 1;
  }
  if (n_cp > n_st) {                                 // the last k-step of an odd K: w0 and xa are its first fragments
    read_x(buf, 0, 0, xb);
    products(w0, xa, 0);
    products(w0, xa, 1);
    products(w0, xb, 0);
    products(w0, xb, 1);
  }
  // factors that the norm left to this kernel (Act::ss): the lane's tokens 32 m + r32
  float rs[MW];
  LmRow lm[MW];
#pragma unroll
  for (int m = 0; m < MW; ++m) rs[m] = 1.f;
  if constexpr (EPI == EPI_LMHEAD) {
#pragma unroll
    for (int m = 0; m < MW; ++m) lm[m] = lm_row(a, tok0 + m * 32 + r32);
  } else if (a.x_ss) {
    f32x4 ss[MW];                                    // all on their way before the first is used
#pragma unroll
    for (int m = 0; m < MW; ++m) ss[m] = row_ss(a, tok0 + m * 32 + r32 < a.T ? tok0 + m * 32 + r32 : 0);
#pragma unroll
    for (int m = 0; m < MW; ++m) rs[m] = row_rstd(a, ss[m]);
  }
  // no copy may outlive the workgroup's LDS, and no fragment read of the last k-step the barrier of the LM head below
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");

  const int nt0 = tw * JW * WR + JW * wr;            // the wave's first weight tile
  if (EPI == EPI_STORE) {
    // lane = weight row r32 of a tile, register q = token 8 (q / 4) + 4 half + q % 4
    float* y = a.y + ((size_t)split * a.T + row_base + tok0) * a.ldy + (size_t)nt0 * 32 + r32;
#pragma unroll
    for (int m = 0; m < MW; ++m)
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int t = m * 32 + 8 * (q >> 2) + 4 * half + (q & 3);
        const float f = a.x_ss ? __shfl(rs[m], t & 31, WAVE) : 1.f;
        if (tok0 + t >= a.T) continue;
#pragma unroll
        for (int j = 0; j < JW; ++j)
          if ((nt0 + j) * 32 + r32 < a.N) y[(size_t)t * a.ldy + 32 * j] = acc[j][m][q] * f;
      }
  } else if (EPI == EPI_SWIGLU) {
    // rows 0..15 of a tile are gate rows, 16..31 the matching up rows: lane (token r32, half) holds features
    // 8 g + 4 half + {0..3}, g = 0, 1, of the tile's sixteen.  The halves trade a group, so that each ends up with
    // eight consecutive features and stores 16 bytes of large terms and 16 of small ones, side by side.
#pragma unroll
    for (int j = 0; j < JW; ++j) {
      const int nt = nt0 + j;
      if (nt >= n_tiles) continue;
#pragma unroll
      for (int m = 0; m < MW; ++m) {
        uint32_t hi[2][2], lo[2][2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float gt = acc[j][m][4 * g + e] * rs[m], up = acc[j][m][4 * (g + 2) + e] * rs[m];
            v[e] = gt / (1.f + __expf(-gt)) * up;
          }
#pragma unroll
          for (int e = 0; e < 2; ++e) split_pair<DT_BF16, 2>(v[2 * e], v[2 * e + 1], hi[g][e], lo[g][e]);
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {                // upper half of group 0 <-> lower half of group 1
          const auto h2 = __builtin_amdgcn_permlane32_swap(hi[0][e], hi[1][e], false, false);
          const auto l2 = __builtin_amdgcn_permlane32_swap(lo[0][e], lo[1][e], false, false);
          hi[0][e] = h2[0]; hi[1][e] = h2[1];
          lo[0][e] = l2[0]; lo[1][e] = l2[1];
        }
        const int t = tok0 + m * 32 + r32;
        if (t < a.T) {
          h16_t* dst = a.act + (size_t)(row_base + t) * a.act_pitch + (size_t)(nt * 2 + half) * 16;
          *reinterpret_cast<u32x4*>(dst) = u32x4{hi[0][0], hi[0][1], hi[1][0], hi[1][1]};
          *reinterpret_cast<u32x4*>(dst + 8) = u32x4{lo[0][0], lo[0][1], lo[1][0], lo[1][1]};
        }
      }
    }
  } else if constexpr (EPI == EPI_LMHEAD) {
    // every wave's copies and fragment reads are complete once it is past this barrier (waves without tokens have left; a
    // barrier counts those that run): the stage buffers become the waves' scratch, a part's weight tiles at a time
    asm volatile("s_barrier" ::: "memory");
    constexpr int JT = TL::LM_TILES;
    f32x4* scr = reinterpret_cast<f32x4*>(lds_raw) + wave * JT * 4 * WAVE;
    const int n_parts = (n_tiles + JT - 1) / JT;
#pragma unroll
    for (int j = 0; j < JW; j += JT)
      if (nt0 + j < n_tiles)
        lmhead_epilogue<JT, MW, false>(a, scr, reinterpret_cast<const f32x16(&)[JT][MW]>(acc[j]), lm, nt0 + j, tok0 >> 5, (nt0 + j) / JT,
                                n_parts, lane);
  }
}

template <int JW, int MW, int WR, int WT, int NB, int EPI>
void launch_form(const GemmArgs& a, int n_wt, int n_tt, int band, hipStream_t st) {
  using TL = LongTiling<JW, MW, WR, WT, NB>;
  static std::once_flag attr_once;                   // raise the dynamic LDS limit once per instantiation, from any thread
  constexpr int lds = EPI == EPI_LMHEAD && TL::LM_SCRATCH > TL::LDS_BYTES ? TL::LM_SCRATCH : TL::LDS_BYTES;
  static_assert(lds <= 160 * 1024, "LDS of a workgroup");
  std::call_once(attr_once, [] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_long_kernel<JW, MW, WR, WT, NB, EPI>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  });
  const long tiles = (long)n_wt * n_tt * a.splits;
  hipLaunchKernelGGL((gemm_long_kernel<JW, MW, WR, WT, NB, EPI>), dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(64 * TL::WAVES),
                     lds, st, a, n_wt, n_tt, band);
}

template <int EPI>
void launch_long(const GemmArgs& a, int form, int n_items, hipStream_t st) {
  const int n_tiles = (a.N + 31) / 32;
  auto tt = [&](int tokens) { return n_items ? n_items : (a.T + tokens - 1) / tokens; };
  auto wt = [&](int rows) { return (n_tiles * 32 + rows - 1) / rows; };
  if (form == LONG_512x128) launch_form<4, 2, 4, 2, 3, EPI>(a, wt(512), tt(128), 4, st);
  else if (form == LONG_128x128) launch_form<2, 2, 2, 2, 3, EPI>(a, wt(128), tt(128), 8, st);
  else if constexpr (EPI != EPI_LMHEAD) {
    if (form == LONG_160x128) launch_form<5, 1, 1, 4, 5, EPI>(a, wt(160), tt(128), 8, st);
    else if (form == LONG_192x128) launch_form<6, 1, 1, 4, 5, EPI>(a, wt(192), tt(128), 8, st);
    else launch_form<4, 2, 4, 1, 2, EPI>(a, wt(512), tt(64), 8, st);     // grouped only
  } else {
    if (form == LONG_320x128) launch_form<5, 1, 2, 4, 4, EPI>(a, wt(320), tt(128), 2, st);
    else launch_form<5, 2, 2, 4, 3, EPI>(a, wt(320), tt(256), 1, st);
  }
}

// Expert-grouped products: 128 rows per tile, or 64 where an expert is not expected to get more than 48 (30B-A3B shape,
// gate/up + down: 32 rows per expert 250 us with tiles of 128, 235 with 64; 64 rows 293 / 350; 1024 rows 2255 / 2476).
// Over the same list, tiles of 128 or 256 weight rows took up to 25 % longer than those of 512 nearly everywhere.
static int grouped_form(int tile_rows) { return tile_rows == 64 ? LONG_512x64 : LONG_512x128; }

}  // namespace

int gemm_long_item_rows(int expected_rows) { return expected_rows <= 48 ? 64 : 128; }

static void fill_long(GemmArgs& a, const Act& x, int N, int K, int T) {
  a.x = x.p; a.x_pitch = x.pitch; a.x_ss = x.ss; a.x_eps = x.eps;
  a.N = N; a.K = K; a.T = T;
  a.ksteps_per_split = (K / 16 + 1) / 2 * 2;
  a.splits = 1;
}

hipError_t gemm_long_store(const LinearW& w, const Act& x, int T, float* y, int ldy, const LongPlan& plan, hipStream_t st) {
  GemmArgs a = {};
  fill_long(a, x, w.N, w.K, T);
  for (int i = 0; i < 3; ++i) { a.w[i] = w.seg[i]; a.w_tiles[i] = (w.rows[i] + 31) / 32; }
  a.splits = plan.splits;
  a.ksteps_per_split = ((w.K / 16 + 1) / 2 + plan.splits - 1) / plan.splits * 2;
  a.y = y; a.ldy = ldy;
  launch_long<EPI_STORE>(a, plan.form, 0, st);
  return hipGetLastError();
}

hipError_t gemm_long_swiglu(const h16_t* w_gate_up, int F, int K, const Act& x, int T, const Act& act, int n_units,
                            hipStream_t st) {
  GemmArgs a = {};
  fill_long(a, x, 2 * F, K, T);
  a.w[0] = w_gate_up; a.w_tiles[0] = F / 16;
  a.act = act.p; a.act_pitch = act.pitch;
  launch_long<EPI_SWIGLU>(a, long_plan(2 * F, K, T, 1, n_units, false).form, 0, st);
  return hipGetLastError();
}

hipError_t gemm_long_grouped_swiglu(const h16_t* w_gate_up, int F, int K, const Act& x, const int32_t* x_rows,
                                    const int32_t* group_off, const Act& act, const GroupItems& items, hipStream_t st) {
  GemmArgs a = {};
  fill_long(a, x, 2 * F, K, 0);
  a.x_rows = x_rows;
  a.w[0] = w_gate_up; a.w_tiles[0] = F / 16; a.w_expert_stride = packed_weight_elems(2 * F, K);
  a.act = act.p; a.act_pitch = act.pitch;
  a.group_off = group_off; a.item_expert = items.expert; a.item_tile = items.tile; a.n_items = items.count;
  launch_long<EPI_SWIGLU>(a, grouped_form(items.tile_rows), items.max_items, st);
  return hipGetLastError();
}

hipError_t gemm_long_grouped_store(const h16_t* w, int N, int K, const Act& x, const int32_t* group_off, float* y,
                                   const GroupItems& items, hipStream_t st) {
  GemmArgs a = {};
  fill_long(a, x, N, K, 0);
  a.w[0] = w; a.w_tiles[0] = (N + 31) / 32; a.w_expert_stride = packed_weight_elems(N, K);
  a.y = y; a.ldy = N;
  a.group_off = group_off; a.item_expert = items.expert; a.item_tile = items.tile; a.n_items = items.count;
  launch_long<EPI_STORE>(a, grouped_form(items.tile_rows), items.max_items, st);
  return hipGetLastError();
}

// The form is long_lmhead_form's.  With 320 x 128 or 320 x 256 in place of 128 x 128, 151 936 ids, one draw per row, us with the
// parts' merge (10 -> 8.5 of it): K 2560, 96 rows 229 -> 207, 128 238 -> 224, 129 359 -> 310, 256 407 -> 374; K 2048, 256 rows 339 -> 316.
// (Of 64 rows and fewer tiles of 160 to 320 rows, one or two workgroups per unit, gave what the short forms give.)
hipError_t gemm_long_lmhead(const h16_t* w_lm, int V, int K, const Act& x, int T, float* logits, float* part,
                            const uint64_t* seeds, const float* temperature, const int32_t* sample_pos,
                            const int32_t* row_seq, bool draw, int n_units, hipStream_t st) {
  GemmArgs a = {};
  fill_long(a, x, V, K, T);
  a.w[0] = w_lm; a.w_tiles[0] = (V + 31) / 32;
  a.logits = logits; a.part = part; a.seeds = seeds; a.temperature = temperature; a.sample_pos = sample_pos;
  a.row_seq = row_seq; a.draw = draw ? 1 : 0;
  launch_long<EPI_LMHEAD>(a, long_lmhead_form(V, K, T, n_units), 0, st);
  return hipGetLastError();
}

}  // namespace rlx
