// GEMM of short calls of dense policies (decode steps, chunks of up to 128 tokens): a wave walks its own part of K alone.
//
//   y[t, n] = sum_k x[t, k] * W[n, k]        fp32 accumulate
//
// A workgroup of four waves owns RT tiles of 16 weight rows and all NT tiles of 16 tokens over its K range, and deals the k-steps
// (32 wide, MFMA 16x16x32) to its waves in turn.  A wave loads the weight and activation fragments of its steps from global
// memory straight into registers, D steps ahead: every byte enters the compute unit once, nothing passes through LDS and no
// barrier couples the waves while they stream.  At the end their sums are added through LDS in wave order.
// What bounds it: with one token tile the weights at the card's rate, with many the ~45 bytes/ns that a compute unit takes in,
// weights and activations together, so the tile is chosen for equal bytes on every unit: 16-row tiles cut the 4B shape's gate/up
// into 244 workgroups of 80 rows where 32-row tiles left 152 of 128 rows.  Two steps ahead are enough (four waves x 13 KB), and
// more were slower everywhere but in the smallest form (us at 45 tokens, D = 2 / 3 / 4: gate/up 22.5 / 23.0 / 22.9, down
// 12.8 / 14.1 / 14.3, o 7.7 / 8.1 / 8.5); eight waves with D = 1 or 2 the same or slower.
// us per launch at the 4B shape, the skinny form -> this one (bf16 in two terms, weights from memory):
//   tokens          1             45            64            96            128
//   gate/up   24.2 -> 17.7  29.7 -> 22.6  32.0 -> 25.4  53.1 -> 31.6  54.8 -> 38.0
//   q|k|v      9.8 ->  7.5  10.9 -> 10.4  11.5 -> 11.9  17.5 -> 15.4  (17.9 -> 19.2)   with two fifths fewer planes
//   o          7.1 ->  5.7   9.3 ->  7.7   9.8 ->  8.6  12.8 -> 11.2  (13.4 -> 14.0)
//   down      12.7 ->  9.8  15.4 -> 12.8  15.8 -> 14.5  24.5 -> 19.1  (25.2 -> 23.4)
//   LM head    128 ->  115
// Calls of few tokens (NORM) make their rows themselves, see below.
#include <mutex>
#include <type_traits>

#include "gemm_core.h"

namespace rlx {
namespace {

template <int RT, int NT, int PL, int EPI>
struct FlowTiling {
  static constexpr int TILES = RT * NT, LOADS = RT + NT * PL;
  static constexpr int D = LOADS <= 4 ? 4 : 2;                             // steps loaded ahead
  static constexpr int NR = TILES <= 32 ? FLOW_WAVES : FLOW_WAVES / 2;     // waves whose sums are in LDS at a time
  typedef std::conditional_t<EPI == EPI_LMHEAD, LmRow, float> PerToken;    // behind the sums: what the epilogue knows of a token
  static constexpr int SUM_BYTES = TILES * NR * 1024, LDS_BYTES = SUM_BYTES + 16 * NT * (int)sizeof(PerToken);
  static_assert(SUM_BYTES % alignof(PerToken) == 0 && LDS_BYTES <= 160 * 1024, "LDS of a workgroup");
};

// Loads by buffer descriptor: uniform base, uniform offset of the step, 32-bit lane offset.  A lane whose offset lies past the
// descriptor's end reads zeros and touches no memory, which serves steps past the end, the missing half of an odd last step
// and token rows past the last one.
constexpr uint32_t NOWHERE = 0x80000000u;            // past the end of every descriptor
typedef __amdgpu_buffer_rsrc_t Desc;
__device__ __forceinline__ Desc make_desc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00027000);
}
template <int AUX>
__device__ __forceinline__ u32x4 desc_load(Desc d, uint32_t lane, uint32_t step) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(d, (int)lane, (int)step, AUX));
}

// ---- LM head: sums of a lane's vocabulary rows ----
// (The steps are those of lmhead_epilogue; as functions that both used they made its loop, 2 to 4 % of a long LM head, slower.  A
// change of one is made in both: the tests hold 1 to 18 rows, in one form and the other, to the same draws.)
struct LmSums { float mx = -INFINITY, se = 0.f, best = -INFINITY; int besti = 0x7FFFFFFF; };
__device__ __forceinline__ float lm_scale(const LmRow& r) { return r.temperature > 0.f ? 1.f / r.temperature : 1.f; }
// uniform over the launch when draw == 0
__device__ __forceinline__ bool lm_draws(const GemmArgs& a, const LmRow& r) { return a.draw != 0 && r.temperature > 0.f; }
// four vocabulary rows nrow .. nrow + 3 (nrow a multiple of 4, below N) of token t: logits v; invt and draw are the row's
// lm_scale() and lm_draws()
__device__ __forceinline__ void lm_add(const GemmArgs& a, LmSums& s, const f32x4& v, int t, int nrow, const LmRow& row, float invt,
                                       bool draw) {
  if (a.logits) {
    if (nrow + 3 < a.N) {
      *reinterpret_cast<f32x4*>(a.logits + (size_t)t * a.N + nrow) = v;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (nrow + j < a.N) a.logits[(size_t)t * a.N + nrow + j] = v[j];
    }
  }
  float z[4], sc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) z[j] = sc[j] = nrow + j < a.N ? v[j] * invt : -INFINITY;
  if (a.draw) {
    uint32_t rnd[4];                                          // one Philox block covers the four ids
    philox4x32_10((uint32_t)(nrow >> 2), row.pos, 0u, 0u, (uint32_t)row.seed, (uint32_t)(row.seed >> 32), rnd);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float noise = gumbel_from_u32(rnd[j]);
      asm volatile("" : "+v"(noise));                         // computed for all lanes: no branch per id
      sc[j] = draw ? z[j] + noise : z[j];
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (sc[j] > s.best) { s.best = sc[j]; s.besti = nrow + j; }   // ascending ids: ties keep the smaller one
  const float nm = fmaxf(s.mx, fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3])));
  s.se = s.se * __expf(s.mx - nm) + ((__expf(z[0] - nm) + __expf(z[1] - nm)) + (__expf(z[2] - nm) + __expf(z[3] - nm)));
  s.mx = nm;
}
// merge with the lane `mask` apart that holds other rows of the same token; both end up with the same bits
__device__ __forceinline__ void lm_merge_lanes(LmSums& s, int mask, bool upper) {
  const float omx = __shfl_xor(s.mx, mask, WAVE), ose = __shfl_xor(s.se, mask, WAVE);
  const float obest = __shfl_xor(s.best, mask, WAVE);
  const int obesti = __shfl_xor(s.besti, mask, WAVE);
  if (obest > s.best || (obest == s.best && obesti < s.besti)) { s.best = obest; s.besti = obesti; }
  const float nm = fmaxf(s.mx, omx);
  if (nm > -INFINITY) {
    // fixed operand order: lower lanes first
    const float lo_m = upper ? omx : s.mx, lo_s = upper ? ose : s.se, hi_m = upper ? s.mx : omx, hi_s = upper ? s.se : ose;
    s.se = lo_s * (lo_m == -INFINITY ? 0.f : __expf(lo_m - nm)) + hi_s * (hi_m == -INFINITY ? 0.f : __expf(hi_m - nm));
    s.mx = nm;
  }
}
__device__ __forceinline__ void lm_store(const GemmArgs& a, const LmSums& s, int t, int part, int n_parts) {
  const f32x4 pv = {s.mx, s.se, s.best, __int_as_float(s.besti)};
  *reinterpret_cast<f32x4*>(a.part + ((size_t)t * n_parts + part) * 4) = pv;
}

// ---- the norm of the rows, where a call has so few of them that every workgroup can make them all (NORM) ----
// A norm kernel costs its launch, a round trip for its row and another for the product's workgroups that wait for it: 3.9 us
// before a product of 8 to 18 at one token.  Here the row's residual and planes (40 KB at the 4B shape) are asked for first and the
// first weights right behind them, so that the norm passes in the shadow of the weights' latency; the rows stay in LDS, one
// 16-byte read per lane, step and term.  The price is the rows and planes once per workgroup, which is what bounds the number of tokens
// (flow_norm_form): up to NV float4 slices of the rows per thread (a step of eight layers of the 4B shape, us: 1 token, three slices
// 638 -> 594; 2, five 670 -> 643; 3, eight 690 -> 700; 4, ten 693 -> 722; the two-layer policy, 4 tokens 92 -> 79).
template <int PL, int EPI>
struct FlowRows {
  // rows that keep their common factor out (Act::ss) but for LM heads, whose rows are read again, and one fp16 term, whose range
  // unnormalised rows would strain
  static constexpr bool LATE_FACTOR = EPI != EPI_LMHEAD && PL == 2;
  __host__ __device__ static int pitch(int K) { return (K + 31) / 32 * 32 + 8; }   // elements; 16 bytes past the banks' period
  __host__ __device__ static int x_bytes(int T, int K) { return PL * T * pitch(K) * 2; }
  // + squares of the slices, + factors
  __host__ __device__ static int bytes(int T, int K) { return x_bytes(T, K) + T * (K / 4) * 4 + FLOW_NORM_ROWS * 4; }
  // ... at most, of calls that fit (flow_norm_fits): so many slices of four elements, and rows that end inside a 32-wide step
  static constexpr int SLICES = FLOW_NORM_NV * 256, MOST = PL * (4 * SLICES + FLOW_NORM_ROWS * 24) * 2 + SLICES * 4 + FLOW_NORM_ROWS * 4;
};
template <int NV, int PL, int FMT, int EPI>
__device__ __forceinline__ void flow_rows_load(const GemmArgs& a, f32x4 (&v)[NV], u32x2 (&gain)[NV]) {
  constexpr int PR = 4;                              // planes per round
  const int nv = a.K >> 2, total = a.T * nv, tid = (int)threadIdx.x;
  __builtin_assume(total > 0);                       // offsets that are not negative: fewer instructions before the first load
  const FlowNorm& m = a.norm;
  int f[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    f[j] = min(256 * j + tid, total - 1);            // a slice past the end repeats the last one and is never stored
    v[j] = *reinterpret_cast<const f32x4*>(m.h + 4 * (size_t)f[j]);
    gain[j] = *reinterpret_cast<const u32x2*>(m.gain + 4 * (f[j] % nv));
  }
  if (!m.add) return;
  for (int s0 = 0; s0 < m.n_planes; s0 += PR) {      // in plane order
    f32x4 p[PR][NV];
#pragma unroll
    for (int q = 0; q < PR; ++q) {
      const size_t plane = (size_t)min(s0 + q, m.n_planes - 1) * a.T * a.K;
#pragma unroll
      for (int j = 0; j < NV; ++j) p[q][j] = *reinterpret_cast<const f32x4*>(m.add + plane + 4 * (size_t)f[j]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < PR; ++q)
      if (s0 + q < m.n_planes) {
#pragma unroll
        for (int j = 0; j < NV; ++j) v[j] += p[q][j];
      }
  }
}
// the rows into LDS as 16-bit terms [term][row][pitch], zeros behind K; the factors that are left out go to `late`
template <int NV, int PL, int FMT, int EPI>
__device__ __forceinline__ void flow_rows_finish(const GemmArgs& a, const f32x4 (&v)[NV], const u32x2 (&gain)[NV], unsigned char* lds,
                                                 float* late, int wg, int n_wgs) {
  using FR = FlowRows<PL, EPI>;
  const int nv = a.K >> 2, total = a.T * nv, tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6, pitch = FR::pitch(a.K);
  h16_t* x = reinterpret_cast<h16_t*>(lds);
  float* sq = reinterpret_cast<float*>(lds + FR::x_bytes(a.T, a.K));
  float* factor = FR::LATE_FACTOR ? late : sq + total;
  const FlowNorm& m = a.norm;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int f = 256 * j + tid;
    if (f >= total) continue;
    sq[f] = v[j][0] * v[j][0] + v[j][1] * v[j][1] + v[j][2] * v[j][2] + v[j][3] * v[j][3];
    if (m.add && m.h_out && j % n_wgs == wg) *reinterpret_cast<f32x4*>(m.h_out + 4 * (size_t)f) = v[j];
  }
  for (int i = tid; i < PL * a.T * (pitch - a.K) / 2; i += 256) {   // zeros behind the rows' ends
    const int w = (pitch - a.K) / 2;
    reinterpret_cast<uint32_t*>(x + (size_t)(i / w) * pitch + a.K)[i % w] = 0u;
  }
  auto put = [&]() {
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int f = 256 * j + tid;
      if (f >= total) continue;
      const int t = f / nv, k = 4 * (f - t * nv);
      const float r = FR::LATE_FACTOR ? 1.f : factor[t];
      float o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float g = h16_to_f32<FMT>((h16_t)((gain[j][e >> 1] >> (16 * (e & 1))) & 0xFFFFu));
        o[e] = FR::LATE_FACTOR ? v[j][e] * g : v[j][e] * r * g;
      }
      uint32_t hi[2], lo[2] = {0u, 0u};
#pragma unroll
      for (int e = 0; e < 2; ++e) split_pair<FMT, PL>(o[2 * e], o[2 * e + 1], hi[e], lo[e]);
      *reinterpret_cast<u32x2*>(x + (size_t)t * pitch + k) = u32x2{hi[0], hi[1]};
      if (PL == 2) *reinterpret_cast<u32x2*>(x + (size_t)(a.T + t) * pitch + k) = u32x2{lo[0], lo[1]};
      if (EPI == EPI_LMHEAD && j % n_wgs == wg) {
        h16_t* dst = m.x_out + frag_act_offset(t, k & ~7, 0, a.x_mtiles, PL) + (k & 7);
        *reinterpret_cast<u32x2*>(dst) = u32x2{hi[0], hi[1]};
        if (PL == 2) *reinterpret_cast<u32x2*>(dst + 512) = u32x2{lo[0], lo[1]};
      }
    }
  };
  if (FR::LATE_FACTOR) put();
  __syncthreads();
  for (int t = wave; t < a.T; t += FLOW_WAVES) {
    float s = 0.f;
    for (int i = lane; i < nv; i += 64) s += sq[t * nv + i];
    s = wave_sum(s);
    if (lane == 0) factor[t] = 1.0f / sqrtf(s / (float)a.K + m.eps);
  }
  if (!FR::LATE_FACTOR) {
    __syncthreads();
    put();
    __syncthreads();
  }
}

template <int RT, int NT, int PL, int FMT, int EPI, int NORM = 0>
__global__ __launch_bounds__(64 * FLOW_WAVES, 1) void gemm_flow_kernel(GemmArgs a) {
  using TL = FlowTiling<RT, NT, PL, EPI>;
  static_assert(!NORM || NT == 1, "few tokens");
  constexpr int D = TL::D, NW = FLOW_WAVES, NR = TL::NR, NONTEMPORAL = 2;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  f32x4* red = reinterpret_cast<f32x4*>(lds_raw);    // [tile][NR][lane]
  typename TL::PerToken* tok_lds = reinterpret_cast<typename TL::PerToken*>(lds_raw + (NORM ? a.lds_split : TL::SUM_BYTES));   // [16 NT]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15, kg = lane >> 4;
  const int split = blockIdx.y;
  const int KS = a.K >> 4, n_half = ((a.N + 31) >> 5) * 2;   // 16-wide k-steps; row tiles
  const int ht0 = blockIdx.x * RT;

  // ---- this wave's steps: s_b + wave, + 4, ... below s_e; an odd last 16 k is a step whose second half is missing ----
  const int s_b = split * a.ksteps_per_split, s_e = min(s_b + a.ksteps_per_split, (KS + 1) >> 1);
  const int n = (s_e - s_b - wave + NW - 1) / NW;    // may be 0

  // ---- addresses ----
  Desc wd[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    const int ht = min(ht0 + r, n_half - 1);         // a row tile past the end repeats the last one and is never stored
    int lt = ht >> 1;
    const h16_t* base = a.w[0];
    if (lt >= a.w_tiles[0]) {
      lt -= a.w_tiles[0];
      base = a.w[1];
      if (lt >= a.w_tiles[1]) { lt -= a.w_tiles[1]; base = a.w[2]; }
    }
    wd[r] = make_desc(base + packed_tile_offset(lt, KS) + (EPI == EPI_SWIGLU ? 8 : 16) * (ht & 1) * 8, NOWHERE - 1);
  }
  const Desc xd = make_desc(a.x, NOWHERE - 1);
  // row of the tile that the lane holds: 16 consecutive ones, or eight gate rows and the eight up rows that go with them
  const int wrow = EPI == EPI_SWIGLU ? c16 + (c16 & 8) : c16;
  const uint32_t x_kstride = (uint32_t)a.x_mtiles * PL * 1024;           // bytes of 16 k of the activations
  const uint32_t w_lane = (uint32_t)(wrow + 32 * (kg & 1)) * 16 + (uint32_t)(kg >> 1) * (W_KSTRIDE * 2);
  uint32_t x_lane[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int tok = 16 * t + c16;
    x_lane[t] = (uint32_t)(tok >> 5) * (PL * 1024) + (uint32_t)((tok & 31) + 32 * (kg & 1)) * 16 + (uint32_t)(kg >> 1) * x_kstride;
    if (tok >= a.T) x_lane[t] = NOWHERE;
  }
  f32x4 row_v[NORM ? NORM : 1];
  u32x2 row_gain[NORM ? NORM : 1];
  if constexpr (NORM) flow_rows_load<NORM, PL, FMT, EPI>(a, row_v, row_gain);
  // the rows' factors (Act::ss) are requested first of all and settled behind the first steps' loads
  f32x4 ssq = {1.f, 1.f, 1.f, 1.f};
  const bool scaled = NORM ? FlowRows<PL, EPI>::LATE_FACTOR : EPI != EPI_LMHEAD && a.x_ss != nullptr;
  LmRow lm = {};                                     // LM head: of token threadIdx.x
  if (EPI == EPI_LMHEAD) lm = lm_row(a, (int)threadIdx.x);
  if (!NORM && scaled) ssq = row_ss(a, min((int)threadIdx.x, a.T - 1));
  __builtin_amdgcn_sched_barrier(0);

  // Where the activations outweigh the weights the workgroups start at different steps: all of them reading the same lines of
  // the activations at the same time made the 4B shape's step of 64 tokens 2.8 % longer (5325 -> 5175 us; 45 tokens 1.0 %, 96
  // 1.9 %; fp16 120 2.0 %); with fewer activations (fp16 45 tokens, bf16 up to 16) nothing or 0.5 % the other way.
  const int rot = NT * PL >= 4 && n > 0 ? (int)blockIdx.x % n : 0;
  struct Step { u32x4 w[RT], x[NORM ? 1 : NT * PL]; };
  auto load = [&](int i, Step& d) {
    const int s = i < n ? s_b + wave + NW * (i + rot < n ? i + rot : i + rot - n) : s_e;
    const uint32_t gone = (s >= s_e || (2 * s + 1 >= KS && kg >= 2)) ? NOWHERE : 0u;
    const uint32_t ws = (uint32_t)s * (2 * W_KSTRIDE * 2), xs = (uint32_t)s * 2 * x_kstride;
    if constexpr (!NORM) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int p = 0; p < PL; ++p) d.x[t * PL + p] = desc_load<0>(xd, x_lane[t] | gone, xs + p * 1024);
    }
#pragma unroll
    for (int r = 0; r < RT; ++r) d.w[r] = desc_load<NONTEMPORAL>(wd[r], w_lane | gone, ws);
    __builtin_amdgcn_sched_barrier(0);
  };
  f32x4 acc[RT][NT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[r][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  Step st[D];
#pragma unroll
  for (int d = 0; d < D; ++d) load(d, st[d]);
  float rstd = 1.f;
  if constexpr (NORM)
    flow_rows_finish<NORM, PL, FMT, EPI>(a, row_v, row_gain, lds_raw, reinterpret_cast<float*>(tok_lds), (int)(blockIdx.x + gridDim.x * blockIdx.y),
                                         (int)(gridDim.x * gridDim.y));
  else if (scaled) rstd = row_rstd(a, ssq);
  asm volatile("" : "+v"(rstd));
  if (EPI == EPI_LMHEAD) asm volatile("" : "+v"(lm.temperature), "+v"(lm.seed), "+v"(lm.pos));
  __builtin_amdgcn_sched_barrier(0);
  // NORM: the lane's token row and features in LDS (lanes past the last token repeat it: their columns are never stored)
  const int x_pitch = NORM ? FlowRows<PL, EPI>::pitch(a.K) : 0;
  const h16_t* x_lds = reinterpret_cast<const h16_t*>(lds_raw) + (NORM ? min(c16, a.T - 1) * x_pitch + 8 * kg : 0);
  for (int i = 0; i < n; i += D)
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if constexpr (NORM) {
        const bool in = i + d < n;                   // past the end the weights are zeros and so are the rows
        const int s = in ? s_b + wave + NW * (i + d) : 0;
        u32x4 x[PL];
#pragma unroll
        for (int p = 0; p < PL; ++p) {
          x[p] = *reinterpret_cast<const u32x4*>(x_lds + (size_t)p * a.T * x_pitch + 32 * s);
          if (!in) x[p] = u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int p = PL - 1; p >= 0; --p)
#pragma unroll
          for (int r = 0; r < RT; ++r) acc[r][0] = mfma_16x16x32<FMT>(st[d].w[r], x[p], acc[r][0]);
        __builtin_amdgcn_sched_barrier(0);
        load(i + D + d, st[d]);
        continue;
      }
#pragma unroll
      for (int p = PL - 1; p >= 0; --p)              // small term first
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
          for (int t = 0; t < NT; ++t) acc[r][t] = mfma_16x16x32<FMT>(st[d].w[r], st[d].x[NORM ? 0 : t * PL + p], acc[r][t]);
      __builtin_amdgcn_sched_barrier(0);
      load(i + D + d, st[d]);
    }

  // ---- the waves' sums, tile by tile in wave order ----
  if constexpr (NORM) __syncthreads();               // the sums lie where the rows were
  if ((int)threadIdx.x < 16 * NT) {
    if constexpr (EPI == EPI_LMHEAD) tok_lds[threadIdx.x] = lm;
    else if (scaled && !NORM) tok_lds[threadIdx.x] = rstd;
  }
  auto put = [&]() {
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int t = 0; t < NT; ++t) red[((r * NT + t) * NR + (wave % NR)) * WAVE + lane] = acc[r][t];
  };
  if (NR < NW) {                                     // LDS holds half: the upper waves hand their sums to the lower ones first
    if (wave >= NR) put();
    __syncthreads();
    if (wave < NR) {
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[r][t] += red[((r * NT + t) * NR + wave) * WAVE + lane];
      put();
    }
  } else {
    put();
  }
  __syncthreads();
  auto sum_of = [&](int tile) {
    f32x4 v = red[tile * NR * WAVE + lane];
#pragma unroll
    for (int w = 1; w < NR; ++w) v += red[(tile * NR + w) * WAVE + lane];
    return v;
  };
  if constexpr (EPI == EPI_LMHEAD) {
    // a part is 32 vocabulary rows, two row tiles: lane = token c16 of the token tile, rows 4 kg .. 4 kg + 3 of each
    static_assert(RT % 2 == 0, "whole parts");
    const int n_parts = n_half / 2;
    for (int p = wave; p < TL::TILES / 2; p += NW) {
      const int part = ht0 / 2 + p / NT, tt = p % NT, t = 16 * tt + c16;
      if (part >= n_parts) break;                    // uniform
      LmSums s;
      if (t < a.T) {
        const LmRow row = tok_lds[t];
        const float invt = lm_scale(row);
        const bool draw = lm_draws(a, row);
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
          const int nrow = 32 * part + 16 * h + 4 * kg;
          if (nrow < a.N) lm_add(a, s, sum_of((2 * (p / NT) + h) * NT + tt), t, nrow, row, invt, draw);
        }
      }
      lm_merge_lanes(s, 16, kg & 1);
      lm_merge_lanes(s, 32, kg >> 1);
      if (t < a.T && kg == 0) lm_store(a, s, t, part, n_parts);
    }
    return;
  }
  for (int tile = wave; tile < TL::TILES; tile += NW) {
    f32x4 v = sum_of(tile);
    const int ht = ht0 + tile / NT, t = 16 * (tile % NT) + c16;
    if constexpr (EPI != EPI_LMHEAD) {
      if (scaled) v *= tok_lds[16 * (tile % NT) + c16];
    }
    if (ht >= n_half) continue;
    if (EPI == EPI_STORE) {
      const int nrow = 16 * ht + 4 * kg;
      float* dst = a.y + ((size_t)split * a.T + t) * a.ldy + nrow;
      if (t < a.T) {
        if (nrow + 3 < a.N) {
          *reinterpret_cast<f32x4*>(dst) = v;
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (nrow + j < a.N) dst[j] = v[j];
        }
      }
    } else {
      // lanes 0..31 hold gate rows 4 (kg & 1) + {0..3}, lanes 32..63 the up rows of the same features: the halves trade, so
      // that the lower lanes hold both of features 0 and 1 of the four and the upper lanes both of features 2 and 3
      const auto e0 = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[0]), __float_as_uint(v[2]), false, false);
      const auto e1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[1]), __float_as_uint(v[3]), false, false);
      const float g0 = __uint_as_float(e0[0]), u0 = __uint_as_float(e0[1]);
      const float g1 = __uint_as_float(e1[0]), u1 = __uint_as_float(e1[1]);
      uint32_t hi, lo = 0;
      split_pair<FMT, PL>(g0 / (1.f + __expf(-g0)) * u0, g1 / (1.f + __expf(-g1)) * u1, hi, lo);
      if (t < a.T && 8 * ht < (a.N >> 1)) {
        h16_t* dst = a.act + frag_act_offset(t, 8 * ht, 0, a.act_mtiles, PL) + 4 * (kg & 1) + 2 * (kg >> 1);
        *reinterpret_cast<uint32_t*>(dst) = hi;
        if (PL == 2) *reinterpret_cast<uint32_t*>(dst + 512) = lo;
      }
    }
  }
}

template <int RT, int NT, int PL, int FMT, int EPI>
void launch_flow_one(const GemmArgs& a, dim3 grid, hipStream_t st) {
  static std::once_flag attr_once;                   // raise the dynamic LDS limit once per instantiation, from any thread
  constexpr int lds = FlowTiling<RT, NT, PL, EPI>::LDS_BYTES;
  std::call_once(attr_once, [] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_flow_kernel<RT, NT, PL, FMT, EPI>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  });
  hipLaunchKernelGGL((gemm_flow_kernel<RT, NT, PL, FMT, EPI>), grid, dim3(64 * FLOW_WAVES), lds, st, a);
}
template <int RT, int PL, int FMT, int EPI, int NORM>
void launch_flow_norm(GemmArgs a, dim3 grid, hipStream_t st) {
  using TL = FlowTiling<RT, 1, PL, EPI>;
  static_assert(FlowRows<PL, EPI>::MOST + 16 <= 60 * 1024 && TL::LDS_BYTES <= 60 * 1024, "below the limit that has to be raised");
  const int rows = (FlowRows<PL, EPI>::bytes(a.T, a.K) + 15) / 16 * 16;
  a.lds_split = rows > TL::SUM_BYTES ? rows : TL::SUM_BYTES;
  hipLaunchKernelGGL((gemm_flow_kernel<RT, 1, PL, FMT, EPI, NORM>), grid, dim3(64 * FLOW_WAVES),
                     a.lds_split + TL::LDS_BYTES - TL::SUM_BYTES, st, a);
}
template <int RT, int NT, int EPI>
void launch_flow_fmt(const GemmArgs& a, dim3 grid, const Act& x, hipStream_t st) {
  if constexpr (NT == 1) {
    if (a.norm.h) {
      const bool few = a.T * (a.K / 4) <= 3 * 256;
      if (x.dtype == DT_F16) few ? launch_flow_norm<RT, 1, DT_F16, EPI, 3>(a, grid, st) : launch_flow_norm<RT, 1, DT_F16, EPI, FLOW_NORM_NV>(a, grid, st);
      else few ? launch_flow_norm<RT, 2, DT_BF16, EPI, 3>(a, grid, st) : launch_flow_norm<RT, 2, DT_BF16, EPI, FLOW_NORM_NV>(a, grid, st);
      return;
    }
  }
  if (x.dtype == DT_F16) launch_flow_one<RT, NT, 1, DT_F16, EPI>(a, grid, st);
  else launch_flow_one<RT, NT, 2, DT_BF16, EPI>(a, grid, st);
}
template <int RT, int EPI>
void launch_flow(const GemmArgs& a, int splits, const Act& x, hipStream_t st) {
  const dim3 grid((((a.N + 31) / 32) * 2 + RT - 1) / RT, splits);
  if (a.T <= 16) launch_flow_fmt<RT, 1, EPI>(a, grid, x, st);
  else if (a.T <= 32) launch_flow_fmt<RT, 2, EPI>(a, grid, x, st);
  else if (a.T <= 48) launch_flow_fmt<RT, 3, EPI>(a, grid, x, st);
  else if (a.T <= 64) launch_flow_fmt<RT, 4, EPI>(a, grid, x, st);
  else if constexpr (RT <= FLOW_RT_MANY) {
    if (a.T <= 96) launch_flow_fmt<RT, 6, EPI>(a, grid, x, st);
    else if constexpr (EPI == EPI_SWIGLU) launch_flow_fmt<RT, 8, EPI>(a, grid, x, st);
    else launch_flow_one<RT, 8, 1, DT_F16, EPI>(a, grid, st);   // stores of two terms end at 96 tokens
  }
}

GemmArgs flow_args(const Act& x, int N, int K, int T, int splits) {
  GemmArgs a = {};
  a.x = x.p; a.x_mtiles = x.mtiles(); a.x_ss = x.ss; a.x_eps = x.eps;
  a.N = N; a.K = K; a.T = T;
  a.ksteps_per_split = ((K / 16 + 1) / 2 + splits - 1) / splits;         // 32-wide steps
  return a;
}
bool flow_format(int planes, int dtype) { return (dtype == DT_BF16 && planes == 2) || (dtype == DT_F16 && planes == 1); }

}  // namespace

static bool norm_fits(const FlowNorm* norm, int T, int K) { return !norm || flow_norm_fits(T, K); }

bool gemm_flow_store_form(int N, int K, int T, int n_units, int planes, int dtype) {
  return flow_format(planes, dtype) && flow_store_form(N, K, T, n_units, planes);
}
hipError_t gemm_flow_store(const LinearW& w, const Act& x, int T, float* y, int ldy, const FlowPlan& plan, hipStream_t st,
                           const FlowNorm* norm) {
  if (!norm_fits(norm, T, w.K)) return hipErrorInvalidValue;
  if (!flow_format(x.planes, x.dtype) || x.pitch || T > (x.planes == 1 ? 128 : 96) || (T > 64 && plan.rt > FLOW_RT_MANY))
    return hipErrorInvalidValue;
  GemmArgs a = flow_args(x, w.N, w.K, T, plan.splits);
  for (int i = 0; i < 3; ++i) { a.w[i] = w.seg[i]; a.w_tiles[i] = (w.rows[i] + 31) / 32; }
  a.y = y; a.ldy = ldy;
  if (norm) a.norm = *norm;
  if (plan.rt == 2) launch_flow<2, EPI_STORE>(a, plan.splits, x, st);
  else if (plan.rt == 4) launch_flow<4, EPI_STORE>(a, plan.splits, x, st);
  else if (plan.rt == 5) launch_flow<5, EPI_STORE>(a, plan.splits, x, st);
  else if (plan.rt == 8) launch_flow<8, EPI_STORE>(a, plan.splits, x, st);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

bool gemm_flow_swiglu_form(int F, int T, int n_units, int planes, int dtype) {
  return flow_format(planes, dtype) && T <= 128 && flow_swiglu_rt(F, T, n_units) > 0;
}
hipError_t gemm_flow_swiglu(const h16_t* w_gate_up, int F, int K, const Act& x, int T, const Act& act, int n_units, hipStream_t st,
                            const FlowNorm* norm) {
  if (!norm_fits(norm, T, K)) return hipErrorInvalidValue;
  if (!gemm_flow_swiglu_form(F, T, n_units, x.planes, x.dtype) || x.pitch || act.pitch) return hipErrorInvalidValue;
  GemmArgs a = flow_args(x, 2 * F, K, T, 1);
  a.w[0] = w_gate_up; a.w_tiles[0] = F / 16;
  a.act = act.p; a.act_mtiles = act.mtiles();
  if (norm) a.norm = *norm;
  const int rt = flow_swiglu_rt(F, T, n_units);
  if (rt == 2) launch_flow<2, EPI_SWIGLU>(a, 1, x, st);
  else if (rt == 4) launch_flow<4, EPI_SWIGLU>(a, 1, x, st);
  else if (rt == 5) launch_flow<5, EPI_SWIGLU>(a, 1, x, st);
  else if (rt == 6) launch_flow<6, EPI_SWIGLU>(a, 1, x, st);
  else launch_flow<8, EPI_SWIGLU>(a, 1, x, st);
  return hipGetLastError();
}

// LM heads of one token tile (151 936 x 2560, 1 token: 128 us in the skinny form, 115 in this one; of more, where the activations
// weigh as much as the weights and the sums through LDS more: 45 tokens in fp16 157 and 171, 64 in bf16 170 and 196)
bool gemm_flow_lmhead_form(int T, int planes, int dtype) { return flow_format(planes, dtype) && T <= 16; }
hipError_t gemm_flow_lmhead(const h16_t* w_lm, int V, int K, const Act& x, int T, float* logits, float* part, const uint64_t* seeds,
                            const float* temperature, const int32_t* sample_pos, const int32_t* row_seq, bool draw, hipStream_t st,
                            const FlowNorm* norm) {
  if (!norm_fits(norm, T, K)) return hipErrorInvalidValue;
  if (!gemm_flow_lmhead_form(T, x.planes, x.dtype) || x.pitch || x.ss) return hipErrorInvalidValue;
  GemmArgs a = flow_args(x, V, K, T, 1);
  a.w[0] = w_lm; a.w_tiles[0] = (V + 31) / 32;
  a.logits = logits; a.part = part; a.seeds = seeds; a.temperature = temperature; a.sample_pos = sample_pos;
  a.row_seq = row_seq; a.draw = draw ? 1 : 0;
  if (norm) { a.norm = *norm; a.norm.x_out = x.p; }
  launch_flow_fmt<8, 1, EPI_LMHEAD>(a, dim3(((V + 31) / 32 * 2 + 7) / 8), x, st);
  return hipGetLastError();
}

}  // namespace rlx
