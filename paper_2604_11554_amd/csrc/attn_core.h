// Pieces shared by the prefill and decode attention kernels (gfx950, MFMA 16x16x32 on bf16 or fp16 operands;
// FMT names the format of the pool and of the query / probability terms).
//
// Pool page of one (layer, block, kv head):  K[16 tokens][hd]  then  V^T[hd][16 tokens].
// The transposed V page makes both contractions read 8 or 16 contiguous bytes per lane:
//   S^T[token, col]  = K[token, :] . Q[col, :]          A = K page rows,  B = Q columns
//   O^T[d, col]     += V^T[d, tokens] . P[tokens, col]  A = V^T rows,     B = P (registers of S^T)
// A "column" is one (query position, query head).  The softmax statistics of a column live in
// the lanes that hold that column, so rescaling is lane-local; the max over keys is reduced
// across the four 16-lane groups with two shuffles.
#pragma once
#include "kernels.h"

namespace rlx {

__device__ __forceinline__ h16x8 load_2x4(const h16_t* p0, const h16_t* p1) {
  u32x2 a = *reinterpret_cast<const u32x2*>(p0);
  u32x2 b = *reinterpret_cast<const u32x2*>(p1);
  u32x4 v = {a[0], a[1], b[0], b[1]};
  return __builtin_bit_cast(h16x8, v);
}
// the same from pages that the launch reads once (decode attention)
__device__ __forceinline__ h16x8 load_2x4_stream(const h16_t* p0, const h16_t* p1) {
  u32x2 a = load_stream_8(p0);
  u32x2 b = load_stream_8(p1);
  u32x4 v = {a[0], a[1], b[0], b[1]};
  return __builtin_bit_cast(h16x8, v);
}

// running softmax state of NCT column tiles: lane holds column (lane & 15), rows d = 16 dt + 4 (lane >> 4) + {0..3}
template <int HD, int NCT>
struct WaveState {
  float m[NCT], l[NCT];
  f32x4 o[NCT][HD / 16];
  __device__ __forceinline__ void reset() {
#pragma unroll
    for (int c = 0; c < NCT; ++c) {
      m[c] = -INFINITY; l[c] = 0.f;
#pragma unroll
      for (int dt = 0; dt < HD / 16; ++dt) o[c][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  // sum the four lane groups' partial denominators of each column (once, after the last key)
  __device__ __forceinline__ void finish_denominators() {
#pragma unroll
    for (int c = 0; c < NCT; ++c) {
      l[c] += __shfl_xor(l[c], 16, WAVE);
      l[c] += __shfl_xor(l[c], 32, WAVE);
    }
  }
};

// x wx + y wy in a merge of two states: the product of x is rounded on its own.  Which of the two it is changes the last bit,
// on which near-ties of a MoE policy's routing turn, and left to the compiler it depends on the code around.
__device__ __forceinline__ float weighted_sum(float x, float wx, float y, float wy) { return __builtin_fmaf(y, wy, x * wx); }

// weight of a state with maximum m in a merge whose maximum is `reference`: an empty state weighs nothing
__device__ __forceinline__ float state_weight(float m, float reference) { return m == -INFINITY ? 0.f : __expf(m - reference); }

// largest value of the four lanes that share a column (lanes 16 apart), by swaps of rows and of halves of the wave
__device__ __forceinline__ float column_max(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return fmaxf(__uint_as_float(h[0]), __uint_as_float(h[1]));
}

// One online-softmax step over 32 keys.  The K fragments of two pages (tokens j0*16.. and j1*16..), the V^T fragments of
// the same 32 tokens and the query fragments are in registers or LDS:
//   k0/k1[ks]: page rows (lane & 15), features 32 ks + 8 (lane >> 4) .. +8
//   vf[dt]:    V^T rows 16 dt + (lane & 15), tokens 4 (lane >> 4) .. +4 of page 0 then of page 1
//   qf(p, c, ks): query fragment of term p, column tile c: column (lane & 15), features 32 ks + 8 (lane >> 4) .. +8
template <int HD, int NCT>
struct Scores { f32x4 a[NCT], b[NCT]; };              // of the keys of page 0 and of page 1: keys 4 (lane >> 4) + {0..3}

template <int HD, int NCT, int PL, int FMT, typename QF>
__device__ __forceinline__ void qk_step(Scores<HD, NCT>& s, const h16x8 (&k0)[HD / 32], const h16x8 (&k1)[HD / 32], QF qf) {
#pragma unroll
  for (int c = 0; c < NCT; ++c) { s.a[c] = f32x4{0.f, 0.f, 0.f, 0.f}; s.b[c] = f32x4{0.f, 0.f, 0.f, 0.f}; }
#pragma unroll
  for (int ks = 0; ks < HD / 32; ++ks)
#pragma unroll
    for (int c = 0; c < NCT; ++c)
#pragma unroll
      for (int p = PL - 1; p >= 0; --p) {   // small term first
        const h16x8 q = qf(p, c, ks);
        s.a[c] = mfma_16x16x32<FMT>(k0[ks], q, s.a[c]);
        s.b[c] = mfma_16x16x32<FMT>(k1[ks], q, s.b[c]);
      }
}

// -inf for the keys that a column does not see, and scaling: a key is visible to column c when its page is valid,
// key < key_end and key <= pos_col[c]; all_visible (uniform over the wave) says that this holds for every key and column,
// which all but the last steps of a run can tell.  (Scaled behind the branch, the scores are known to be products where their
// maximum is taken, which saves a canonicalising operation per score.)
template <int HD, int NCT>
__device__ __forceinline__ void mask_and_scale(Scores<HD, NCT>& s, int key_base0, int key_base1, bool ok0, bool ok1, int key_end,
                                               const int (&pos_col)[NCT], bool all_visible, float scale, int g) {
#pragma clang fp contract(off)          // the products are rounded on their own, not fused with the softmax's subtraction
  if (!all_visible) {
#pragma unroll
    for (int c = 0; c < NCT; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int key0 = key_base0 + 4 * g + v, key1 = key_base1 + 4 * g + v;
        if (!(ok0 && key0 < key_end && key0 <= pos_col[c])) s.a[c][v] = -INFINITY;
        if (!(ok1 && key1 < key_end && key1 <= pos_col[c])) s.b[c][v] = -INFINITY;
      }
  }
#pragma unroll
  for (int c = 0; c < NCT; ++c) { s.a[c] *= scale; s.b[c] *= scale; }
}

// The vector arithmetic of a step: per score a subtraction, the exponential, an addition and three operations for its
// two terms.  (With compares and selects on every score, the 16-bit conversions in integer operations and the maximum
// through LDS it was about thirty per score, twice the time of the step's 32 matrix products; same bits.)  It leaves
// the weights as B operands and the factor alpha by which the sums so far have to be multiplied before they go on.
template <int HD, int NCT, int PL, int FMT>
__device__ __forceinline__ void softmax_step(WaveState<HD, NCT>& st, const Scores<HD, NCT>& s, h16x8 (&pf)[PL][NCT],
                                             float (&alpha)[NCT]) {
#pragma unroll
  for (int c = 0; c < NCT; ++c) {
    float mx = fmaxf(fmaxf(fmaxf(s.a[c][0], s.a[c][1]), fmaxf(s.a[c][2], s.a[c][3])),
                     fmaxf(fmaxf(s.b[c][0], s.b[c][1]), fmaxf(s.b[c][2], s.b[c][3])));
    mx = column_max(mx);
    const float mn = fmaxf(st.m[c], mx);
    const float ref = mn == -INFINITY ? 0.f : mn;       // a column that has seen no key: every weight below is 0
    alpha[c] = __expf(st.m[c] - ref);
    float p0[4], p1[4], ps = 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      p0[v] = __expf(s.a[c][v] - ref);
      p1[v] = __expf(s.b[c][v] - ref);
      ps += p0[v] + p1[v];
    }
    st.l[c] = st.l[c] * alpha[c] + ps;  // partial over this lane's keys; lane groups are summed at the end
    st.m[c] = mn;
    u32x4 ph, pl;
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      uint32_t h, l = 0;
      split_pair<FMT, PL>(p0[2 * v], p0[2 * v + 1], h, l);
      ph[v] = h; pl[v] = l;
      split_pair<FMT, PL>(p1[2 * v], p1[2 * v + 1], h, l);
      ph[2 + v] = h; pl[2 + v] = l;
    }
    pf[0][c] = ph;
    if (PL == 2) pf[PL - 1][c] = pl;
  }
}

// LATE: past the first thousand keys most steps move no column's maximum, and a factor of 1 leaves the bits as they are.  (Before
// that the branch, which splits the step's instructions into blocks that cannot be interleaved, costs more than it saves.)
template <int HD, int NCT, bool LATE>
__device__ __forceinline__ void rescale(WaveState<HD, NCT>& st, const float (&alpha)[NCT]) {
  if (LATE) {
    bool moved = false;
#pragma unroll
    for (int c = 0; c < NCT; ++c) moved |= alpha[c] != 1.f;
    if (!__builtin_amdgcn_ballot_w64(moved)) return;
  }
#pragma unroll
  for (int c = 0; c < NCT; ++c)
#pragma unroll
    for (int dt = 0; dt < HD / 16; ++dt) st.o[c][dt] *= alpha[c];
}

template <int HD, int NCT, int PL, int FMT>
__device__ __forceinline__ void pv_step(WaveState<HD, NCT>& st, const h16x8 (&vf)[HD / 16], const h16x8 (&pf)[PL][NCT]) {
#pragma unroll
  for (int dt = 0; dt < HD / 16; ++dt)
#pragma unroll
    for (int c = 0; c < NCT; ++c)
#pragma unroll
      for (int p = PL - 1; p >= 0; --p)
        st.o[c][dt] = mfma_16x16x32<FMT>(vf[dt], pf[p][c], st.o[c][dt]);
}

template <int HD, int NCT, int PL, int FMT, bool LATE = false, typename QF>
__device__ __forceinline__ void pair_step(WaveState<HD, NCT>& st, const h16x8 (&k0)[HD / 32],
                                          const h16x8 (&k1)[HD / 32], const h16x8 (&vf)[HD / 16], QF qf,
                                          int key_base0, int key_base1, bool ok0, bool ok1, int key_end,
                                          const int (&pos_col)[NCT], bool all_visible, float scale, int g) {
  Scores<HD, NCT> s;
  h16x8 pf[PL][NCT];
  float alpha[NCT];
  qk_step<HD, NCT, PL, FMT>(s, k0, k1, qf);
  mask_and_scale<HD, NCT>(s, key_base0, key_base1, ok0, ok1, key_end, pos_col, all_visible, scale, g);
  softmax_step<HD, NCT, PL, FMT>(st, s, pf, alpha);
  rescale<HD, NCT, LATE>(st, alpha);
  pv_step<HD, NCT, PL, FMT>(st, vf, pf);
}

// merge the state held in LDS (written by another wave) into this wave's registers
template <int HD, int NCT>
__device__ __forceinline__ void merge_from_lds(WaveState<HD, NCT>& st, const float* ml, const f32x4* ob, int lane) {
#pragma unroll
  for (int c = 0; c < NCT; ++c) {
    float mb = ml[(c * 2 + 0) * WAVE + lane], lb = ml[(c * 2 + 1) * WAVE + lane];
    float mn = fmaxf(st.m[c], mb);
    const float aa = state_weight(st.m[c], mn), ab = state_weight(mb, mn);
    st.l[c] = weighted_sum(lb, ab, st.l[c], aa);
    st.m[c] = mn;
#pragma unroll
    for (int dt = 0; dt < HD / 16; ++dt) {
      const f32x4 v = ob[(c * (HD / 16) + dt) * WAVE + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        st.o[c][dt][e] = dt < 2 ? weighted_sum(st.o[c][dt][e], aa, v[e], ab) : weighted_sum(v[e], ab, st.o[c][dt][e], aa);
    }
  }
}

template <int HD, int NCT>
__device__ __forceinline__ void store_to_lds(const WaveState<HD, NCT>& st, float* ml, f32x4* ob, int lane) {
#pragma unroll
  for (int c = 0; c < NCT; ++c) {
    ml[(c * 2 + 0) * WAVE + lane] = st.m[c];
    ml[(c * 2 + 1) * WAVE + lane] = st.l[c];
#pragma unroll
    for (int dt = 0; dt < HD / 16; ++dt) ob[(c * (HD / 16) + dt) * WAVE + lane] = st.o[c][dt];
  }
}

// Fixed-order tree merge of a workgroup's four waves, (0<-2, 1<-3) then 0<-1; the result is valid in wave 0.
// lds_o: [2][NCT * HD/16 * 64] f32x4, lds_ml: [2][NCT * 2 * 64] floats.  Every wave must call this.
template <int HD, int NCT>
__device__ __forceinline__ void merge_waves(WaveState<HD, NCT>& st, f32x4* lds_o, float* lds_ml, int wave, int lane) {
  constexpr int NO = NCT * (HD / 16) * WAVE, NM = NCT * 2 * WAVE;
  if (wave >= 2) store_to_lds<HD, NCT>(st, lds_ml + (wave - 2) * NM, lds_o + (wave - 2) * NO, lane);
  __syncthreads();
  if (wave < 2) merge_from_lds<HD, NCT>(st, lds_ml + wave * NM, lds_o + wave * NO, lane);
  __syncthreads();
  if (wave == 1) store_to_lds<HD, NCT>(st, lds_ml, lds_o, lane);
  __syncthreads();
  if (wave == 0) merge_from_lds<HD, NCT>(st, lds_ml, lds_o, lane);
}

// Normalised column c of `st` -> 16-bit (hi, lo) terms at row `trow`, features head*HD + ...; every lane of the wave
// calls it (`store` says whether the lane's column exists).  A lane holds four features of every 16-feature tile; lanes
// 16 apart trade those of two tiles, so that each stores whole groups of eight: 16 bytes of large terms, 16 of small ones.
template <int HD, int NCT, int PL, int FMT>
__device__ __forceinline__ void store_column(const WaveState<HD, NCT>& st, int c, const Act& o, int trow, int head,
                                             int g, bool store) {
  const float inv = st.l[c] > 0.f ? 1.f / st.l[c] : 0.f;
#pragma unroll
  for (int dt = 0; dt < HD / 16; dt += 2) {
    uint32_t hi[2][2], lo[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const f32x4 v = st.o[c][dt + i] * inv;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        uint32_t h, l = 0;
        split_pair<FMT, PL>(v[2 * j], v[2 * j + 1], h, l);
        hi[i][j] = h; lo[i][j] = l;
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {                      // odd rows of tile dt <-> even rows of tile dt + 1
      const auto h2 = __builtin_amdgcn_permlane16_swap(hi[0][j], hi[1][j], false, false);
      hi[0][j] = h2[0]; hi[1][j] = h2[1];
      if (PL == 2) {
        const auto l2 = __builtin_amdgcn_permlane16_swap(lo[0][j], lo[1][j], false, false);
        lo[0][j] = l2[0]; lo[1][j] = l2[1];
      }
    }
    // rows 0 and 2 of the wave now hold the two groups of tile dt, rows 1 and 3 those of tile dt + 1
    if (store) {
      h16_t* dst = o.p + o.group_offset(trow, head * HD + 16 * (dt + (g & 1)) + 8 * (g >> 1));
      *reinterpret_cast<u32x4*>(dst) = u32x4{hi[0][0], hi[0][1], hi[1][0], hi[1][1]};
      if (PL == 2) *reinterpret_cast<u32x4*>(dst + o.small_terms()) = u32x4{lo[0][0], lo[0][1], lo[1][0], lo[1][1]};
    }
  }
}

}  // namespace rlx
