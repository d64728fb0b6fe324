// What the GEMM kernels share: their argument block and their epilogues (plain store, SwiGLU, LM head with fused
// log-sum-exp and Gumbel-max partials per 32-row weight tile).
#pragma once
#include "kernels.h"

namespace rlx {

struct GemmArgs {
  const h16_t* x;        // activations [T_x, K]: `PL` terms in fragment order, or rows of two (x_pitch)
  int x_mtiles;           // ceil(T_x / 32)
  const float* x_ss;      // optional: activation row t lacks the factor rstd(t) of its norm (Act::ss); outputs take it
  float x_eps;
  const int32_t* x_rows;  // grouped gate/up: logical row r of the group reads activation row x_rows[r]
  const h16_t* w[3];     // packed weights, up to three stacked row segments
  int w_tiles[3];         // 32-row tiles per segment
  int N, K, T;
  int ksteps_per_split;   // k-steps (16 wide) per blockIdx.y
  float* y;               // EPI_STORE: [splits][T][ldy]
  int ldy;
  h16_t* act;            // EPI_SWIGLU: [act_rows, N / 2], like x (act_pitch)
  int act_mtiles;
  // LM-head epilogue
  float* logits;          // optional [T][N]
  float* part;            // [T][n_parts][4] = max, sumexp, best score, best index (as float bits)
  const uint64_t* seeds;
  const float* temperature;
  const int32_t* sample_pos;
  const int32_t* row_seq;     // optional: row t takes its temperature from entry row_seq[t] (scoring: token -> sequence)
  int draw;                   // 0: no Gumbel-max draw (scoring): the random words are not generated
  // expert-grouped form: blockIdx.y is the expert, its rows are [group_off[e], group_off[e+1])
  const int32_t* group_off;
  size_t w_expert_stride;     // packed elements between consecutive experts' matrices
  // expert-grouped decode form without a grouping pass: the kernel finds its expert's rows in the routing table itself
  const int32_t* route_idx;   // [n_pairs] expert of pair p = token * top_k + slot, or null (rows come from group_off)
  int n_pairs, top_k;
  int n_experts, expert_wgs;  // expert-grouped decode form: experts, and workgroups per expert that has rows
  int32_t* pub_group_off;     // [E + 1] written by this launch: first row of every expert in expert order
  int32_t* pub_pair_pos;      // [n_pairs] written by this launch: row of every pair in expert order
  // long-call form (gemm_long.hip): x is in rows (Act::pitch), and so is act
  size_t x_pitch, act_pitch;
  int splits;                 // K ranges of ksteps_per_split k-steps, a plane of y each
  const int32_t* item_expert; // grouped: expert and row tile of every item, and the number of items (GroupItems)
  const int32_t* item_tile;
  const int32_t* n_items;
  // calls of few tokens (gemm_flow.hip): the kernel makes its rows from the residual stream itself (FlowNorm)
  FlowNorm norm;
  int lds_split;              // where the tokens' entries begin in LDS
};

enum { EPI_STORE = 0, EPI_SWIGLU = 1, EPI_LMHEAD = 2 };

// ---- Philox-4x32-10 (Salmon et al., SC'11), written from the published definition ----
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                              uint32_t k1, uint32_t (&out)[4]) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    uint64_t p0, p1, carry;                          // one instruction for both halves of a product
    asm("v_mad_u64_u32 %0, %1, %2, %3, 0" : "=v"(p0), "=s"(carry) : "v"(c0), "s"(0xD2511F53u));
    asm("v_mad_u64_u32 %0, %1, %2, %3, 0" : "=v"(p1), "=s"(carry) : "v"(c2), "s"(0xCD9E8D57u));
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0, n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
    c0 = n0; c1 = (uint32_t)p1; c2 = n2; c3 = (uint32_t)p0;
    k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
  }
  out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// Gumbel(0,1) from a 32-bit word: u = (R + 0.5) 2^-32, g = -log(-log u).  The largest values of g, the ones that
// win the draw, come from u next to 1: there (1 - u < 2^-6) -log u is taken from w = 1 - u (exact from the integer) by the
// series w + w^2/2 + w^3/3 + w^4/4 (relative error w^4/5 < 2e-8), elsewhere by the hardware's base-2 logarithm (absolute
// error ~1e-7 on a value of at least 0.0156, which is also what the outer logarithm carries): g is within ~1e-5 of the
// exact value, three orders below the tolerance on the scores it is added to.  Two logarithms and a dozen operations,
// branch-free; with a third logarithm and branches around them the four draws of a step cost 5 us in a 17 us LM head.
__device__ __forceinline__ float gumbel_from_u32(uint32_t r) {
  constexpr float LN2 = 0.693147182f;
  const float u = __builtin_fmaf((float)r, 2.3283064365386963e-10f, 1.16415321826934814e-10f);
  const float w = __builtin_fmaf((float)~r, 2.3283064365386963e-10f, 1.16415321826934814e-10f);   // 1 - u
  const float series = w * __builtin_fmaf(w, __builtin_fmaf(w, __builtin_fmaf(w, 0.25f, 0.33333334f), 0.5f), 1.f);
  const float log_u = __builtin_amdgcn_logf(u) * -LN2;           // u >= 2^-33: no subnormal reaches the logarithms
  const float nl = r >= 0xFC000000u ? series : log_u;
  return __builtin_amdgcn_logf(nl) * -LN2;
}

// factor that the norm left out of activation row `tok` (Act::ss): the same expression as in the norm kernel
__device__ __forceinline__ f32x4 row_ss(const GemmArgs& a, int tok) {
  return *reinterpret_cast<const f32x4*>(a.x_ss + (size_t)NORM_PARTS * tok);
}
__device__ __forceinline__ float row_rstd(const GemmArgs& a, const f32x4& p) {
  return 1.0f / sqrtf(((p[0] + p[1]) + (p[2] + p[3])) / (float)a.K + a.x_eps);
}

// Epilogue of one 32-row weight tile `nt` over token tiles mt0 .. mt0 + MT - 1: lane holds token r32 of each token
// tile, rows n0 + 8q + 4*half + {0..3}, q = 0..3, of the accumulators.
// rs[m]: factor of the lane's activation row in token tile m (row_rstd, or 1), fetched by the caller before its main
// loop so that the round trip is not spent at the end of the kernel
template <int MT, int EPI, int PL, int FMT>
__device__ __forceinline__ void tile_epilogue(const GemmArgs& a, const f32x16 (&acc)[MT], int nt, int n_tiles, int mt0,
                                              int split, int row_base, int lane, const float (&rs)[MT]) {
  const int r32 = lane & 31, half = lane >> 5;
  const int n0 = nt * 32;
  if (EPI == EPI_STORE) {
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int t = (mt0 + m) * 32 + r32;
      if (t >= a.T) continue;
      float* dst = a.y + ((size_t)split * a.T + row_base + t) * a.ldy;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int nrow = n0 + 8 * q + 4 * half;
        f32x4 v = {acc[m][4 * q], acc[m][4 * q + 1], acc[m][4 * q + 2], acc[m][4 * q + 3]};
        if (a.x_ss) v *= rs[m];
        if (nrow + 3 < a.N) {
          *reinterpret_cast<f32x4*>(dst + nrow) = v;
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (nrow + j < a.N) dst[nrow + j] = v[j];
        }
      }
    }
  } else if (EPI == EPI_SWIGLU) {
    // The packed matrix interleaves gate and up: rows 0..15 of a tile are gate rows of features
    // 16 nt .. 16 nt + 15, rows 16..31 the matching up rows, so a lane holds both halves of a pair
    // (register groups q and q + 2).  The output feature is the K index of the down projection.
    const int n_feat = a.N >> 1;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int t = (mt0 + m) * 32 + r32;
      if (t >= a.T) continue;
      const int orow = row_base + t;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int feat = nt * 16 + 8 * q + 4 * half;   // four consecutive features inside one 8-group
        if (feat >= n_feat) continue;
        h16_t hi[4], lo[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float g = acc[m][4 * q + j], u = acc[m][4 * (q + 2) + j];
          if (a.x_ss) { g *= rs[m]; u *= rs[m]; }
          split_h16<FMT>(g / (1.f + __expf(-g)) * u, hi[j], lo[j]);
        }
        h16_t* dst = a.act + frag_act_offset(orow, feat & ~7, 0, a.act_mtiles, PL) + (feat & 7);
        u32x2 pk = {(uint32_t)hi[0] | ((uint32_t)hi[1] << 16), (uint32_t)hi[2] | ((uint32_t)hi[3] << 16)};
        *reinterpret_cast<u32x2*>(dst) = pk;
        if (PL == 2) {
          u32x2 pk2 = {(uint32_t)lo[0] | ((uint32_t)lo[1] << 16), (uint32_t)lo[2] | ((uint32_t)lo[3] << 16)};
          *reinterpret_cast<u32x2*>(dst + 512) = pk2;
        }
      }
    }
  }
}

// LM-head epilogue of a wave: per token, its 32 JT vocabulary rows (tiles nt0 ..) are reduced to (max, sumexp, best
// score, its id), record `part` of `n_parts` of the token's row.  The accumulators go through a scratch area in LDS
// (`scr`: JT * 4 KB of the wave's own, one token tile at a time), which lets the work on them run as a loop: written out
// over the registers it was up to 50 KB of straight code per form.  The parts' order of sums differs from a sum id by id, not their
// precision.
// What it needs to know of the lane's row is passed in, so that the caller can ask for it early (three dependent fetches
// at the end of a kernel are three round trips).
struct LmRow { float temperature; uint64_t seed; uint32_t pos; };
__device__ __forceinline__ LmRow lm_row(const GemmArgs& a, int t) {
  const int tc = t < a.T ? t : 0;
  LmRow r = {a.temperature[a.row_seq ? a.row_seq[tc] : tc], 0ull, 0u};
  if (a.draw) { r.seed = a.seeds[tc]; r.pos = (uint32_t)a.sample_pos[tc]; }
  return r;
}
// LINES: how the logits leave (if they are asked for).  In lines of a row, past the caches, eight lanes a line, or by each lane its own
// 16 bytes of a row per instruction, of rows that lie a vocabulary apart.  What the caches hold back they write while other
// workgroups' weights stream: 45 rows of 151 936 ids, K 2560, 174 us -> 158, fp16 157 -> 146 (whole lines alone 171 and 154; no
// logits 157 and 133).  The long-call forms have no other workgroup on the unit that would use the time and pay for the passes through
// LDS: as fast by lanes (151 936 ids with logits, two runs, 5 % apart at most, lanes / lines: K 2560, 128 rows 231, 225 / 223, 228,
// 256 rows 446, 424 / 436, 435; K 2048, 128 rows 198, 187 / 199, 187) or faster (96 rows 168, 167 / 179, 185).
template <int JT, int MT, bool LINES>
__device__ __forceinline__ void lmhead_epilogue(const GemmArgs& a, f32x4* scr, const f32x16 (&acc)[JT][MT], const LmRow (&row)[MT],
                                                int nt0, int mt0, int part, int n_parts, int lane) {
  const int r32 = lane & 31, half = lane >> 5;
#pragma unroll
  for (int m = 0; m < MT; ++m) {
#pragma unroll
    for (int j = 0; j < JT; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        scr[(j * 4 + q) * WAVE + (lane ^ (2 * q + half))] =
            f32x4{acc[j][m][4 * q], acc[j][m][4 * q + 1], acc[j][m][4 * q + 2], acc[j][m][4 * q + 3]};
    if (LINES && a.logits) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // written by other lanes of the wave
      const int c = lane & 7;
#pragma unroll
      for (int j = 0; j < JT; ++j)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int tok = 8 * k + (lane >> 3), tt = (mt0 + m) * 32 + tok, nrow = (nt0 + j) * 32 + 4 * c;
          const f32x4 v = scr[(j * 4 + (c >> 1)) * WAVE + ((tok + 32 * (c & 1)) ^ c)];
          if (tt < a.T && nrow < a.N) {
            float* dst = a.logits + (size_t)tt * a.N + nrow;
            if (nrow + 3 < a.N) {
              __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(dst));
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e)
                if (nrow + e < a.N) dst[e] = v[e];
            }
          }
        }
      asm volatile("" ::: "memory");                       // the next token tile's writes stay behind the other lanes' reads
    }
    const int t = (mt0 + m) * 32 + r32;
    const bool ok = t < a.T;
    float mx = -INFINITY, se = 0.f, best = -INFINITY;
    int besti = 0x7FFFFFFF;
    if (ok) {
      const float temp = row[m].temperature, invt = temp > 0.f ? 1.f / temp : 1.f;
      const bool draw = a.draw != 0 && temp > 0.f;            // uniform over the launch when draw == 0
      const uint64_t seed = row[m].seed;
      const uint32_t pos = row[m].pos;
#pragma unroll 1
      for (int i = 0; i < 4 * JT; ++i) {
        const int nrow = nt0 * 32 + 8 * i + 4 * half;         // multiple of 4: one Philox block covers the four ids
        if (nrow >= a.N) break;
        const f32x4 v = scr[i * WAVE + (lane ^ (2 * (i & 3) + half))];
        if (!LINES && a.logits) {
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
          uint32_t rnd[4];
          philox4x32_10((uint32_t)(nrow >> 2), pos, 0u, 0u, (uint32_t)seed, (uint32_t)(seed >> 32), rnd);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            float noise = gumbel_from_u32(rnd[j]);
            asm volatile("" : "+v"(noise));                     // computed for all lanes: no branch per id
            sc[j] = draw ? z[j] + noise : z[j];
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (sc[j] > best) { best = sc[j]; besti = nrow + j; }   // ascending ids: ties keep the smaller one
        const float nm = fmaxf(mx, fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3])));
        se = se * __expf(mx - nm) + ((__expf(z[0] - nm) + __expf(z[1] - nm)) + (__expf(z[2] - nm) + __expf(z[3] - nm)));
        mx = nm;
      }
    }
    // merge the two half-waves (rows 8i+0..3 and 8i+4..7) of the same token
    const float omx = __shfl_xor(mx, 32, WAVE), ose = __shfl_xor(se, 32, WAVE);
    const float obest = __shfl_xor(best, 32, WAVE);
    const int obesti = __shfl_xor(besti, 32, WAVE);
    if (obest > best || (obest == best && obesti < besti)) { best = obest; besti = obesti; }
    const float nm = fmaxf(mx, omx);
    if (nm > -INFINITY) {
      // fixed operand order (lower half first) so both half-waves compute the same bits
      const float lo_m = half ? omx : mx, lo_s = half ? ose : se, hi_m = half ? mx : omx, hi_s = half ? se : ose;
      se = lo_s * (lo_m == -INFINITY ? 0.f : __expf(lo_m - nm)) + hi_s * (hi_m == -INFINITY ? 0.f : __expf(hi_m - nm));
      mx = nm;
    }
    if (ok && half == 0) {
      const f32x4 pv = {mx, se, best, __int_as_float(besti)};
      *reinterpret_cast<f32x4*>(a.part + ((size_t)t * n_parts + part) * 4) = pv;
    }
  }
}

}  // namespace rlx
