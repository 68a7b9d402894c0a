// bf16 MFMA forward kernels of SSA (paper eq. (4)-(6), Algorithm 1, window paragraph) for gfx950.
//
// Compression and window kernels: a workgroup owns 32 query rows per wavefront = consecutive sorted tokens x
// the h_s heads of one KV group; each wavefront keeps 32 query columns and their softmax state
// (Algorithm 1's m, l, o) in registers.  The selection kernel turns the loops round (per selected block, over the
// tokens that selected it: mfma_slc.hip) with the same tile arithmetic.  Scores are produced TRANSPOSED (S^T = K Q^T, keys x
// queries) so that the probabilities land in the lanes exactly as the B operand of the second contraction O^T = V^T P^T needs them.
// Key tiles (K rows and V rows, both row-major) are staged through LDS once per workgroup (see mfma_t32.h); the K
// operand is one 16-byte LDS read, the V^T operand comes from the same row-major V tile through the transposing
// LDS read of gfx950, so no transposed copy of V exists anywhere.
#include "mfma_common.h"
#include "topk_device.h"
#include "mfma_launch.h"
#include "mfma_qc.h"
#include "mfma_t32.h"
#include "cmp_form.h"
#include "profile.h"

#include <limits.h>
#include <mutex>
#include <type_traits>

namespace {

struct FwdArgs {
  MfmaView v;
  const bf16_t *Q;
  bf16_t *Ob;    // [3,N,Hq,D]
  float *lse;    // [3,N,Hq]
  int32_t *idx;  // [N,Hkv,T]
  float *nlse;   // [N(pos)][Hq]: minus the compression branch's log-sum-exp in log2 units, from m_cmp_walk to m_cmp_scores
  uint32_t *cnt; // [tiles of sorted positions][Hkv*Ns]: m_cmp_fwd adds how many of the tile's tokens selected a block; null: not wanted
};

// Walks start at a multiple of 8 (which keys are a column's first tile, and with it the reference exponent, is part of what the
// selection scores are rounded to).
__device__ inline int walk_begin(int rs) { return rs & ~7; }

// One whole walk of a workgroup over the key range [rs, re) that every column sees.
// False if the sums of some column left the range of the floats (again: a word of LDS, 0).  refs: where the references
// go, in score units (a float per query row of LDS).
template <int D, int NW, class Sum>
__device__ inline bool fwd_walk(T32State<D, Sum> &st, float *refs, const bf16x8 (&qop)[D / 16], const T32Src<2> &src, unsigned char *stage0, int *again,
                                int rs, int re, const typename T32<D, true>::Lanes &ln, float sl2) {
  using T = T32<D, true>;
  t32_clear(st);
  const int first = walk_begin(rs);
  t32_pipeline<D, 2, 64 * NW, 32, std::is_same_v<Sum, SumInOrder>>(src, stage0, first, re, [&](lds_cptr kt, int kb) {
    f32x16 s = t32_scores<D, true>(qop, kt, ln, splat16(0.f));
    if (kb == first || kb + 32 > re) t32_only_keys(s, kb, rs, re);
    if (kb == first) {
      const float raw = t32_column_max(max16(s));
      refs[(threadIdx.x >> 6) * 32 + (threadIdx.x & 31)] = raw;
      st.m = raw * sl2;
    }
    t32_softmax<D, true, false>(st, s, kt + T::BYTES, ln, sl2);
  });
  if (!t32_in_range(st)) *again = 1;
  __syncthreads();
  return !lds_uniform(again);
}

// The walk with a running maximum and a key range [lo, hi) of its own for every column.
template <int D, int NW, class Sum>
__device__ inline void fwd_walk_general(T32State<D, Sum> &st, const bf16x8 (&qop)[D / 16], const T32Src<2> &src, unsigned char *stage0, int rs, int re,
                                        int lo, int hi, const typename T32<D, true>::Lanes &ln, float sl2) {
  t32_clear(st);
  t32_pipeline<D, 2, 64 * NW, 32, std::is_same_v<Sum, SumInOrder>>(src, stage0, walk_begin(rs), re, [&](lds_cptr kt, int kb) {
    f32x16 s = t32_scores<D, true>(qop, kt, ln, splat16(0.f));
    t32_only_keys(s, kb, lo, hi);
    t32_softmax_running<D, true>(st, s, kt + T32<D, true>::BYTES, ln, sl2);
  });
}

// of_pos, start: the range (item, window) of a sorted position and the first key of every range.  True if every
// column saw all keys and its reference is in refs.
template <int D, int NW, class Sum>
__device__ inline bool fwd_branch(T32State<D, Sum> &st, float *refs, const bf16x8 (&qop)[D / 16], const T32Src<2> &src, unsigned char *stage0, int *again,
                                  int rs, int re, bool one, const int32_t *of_pos, const int32_t *start, const MfmaView &v, int wg_pos0,
                                  float sl2) {
  const typename T32<D, true>::Lanes ln = T32<D, true>::lanes();
  if (one && fwd_walk<D, NW>(st, refs, qop, src, stage0, again, rs, re, ln, sl2)) return true;
  const int own = of_pos[query_col(v, wg_pos0, 0).pos];
  fwd_walk_general<D, NW>(st, qop, src, stage0, rs, re, start[own], start[own + 1], ln, sl2);
  return false;
}

// Normalise (Algorithm 1: o * exp(m - l)), store the branch output and its log-sum-exp; returns it in log2 units (the reference
// times the scale and the logarithm added in one rounding where the walk left the reference).
template <int D, class Sum>
__device__ inline float finish(const FwdArgs &a, const T32State<D, Sum> &st, const float *refs, bool have_ref, int branch, const QCol &q) {
  const int h = threadIdx.x >> 5 & 1;
  const float l = st.l.total();
  const float inv = l > 0.f ? 1.0f / l : 0.f;
  float lse2 = l > 0.f ? st.m + __log2f(l) : -INFINITY;
  if (have_ref) lse2 = __builtin_fmaf(refs[(threadIdx.x >> 6) * 32 + (threadIdx.x & 31)], a.v.sl2, __log2f(l));
  if (q.valid) {
    bf16_t *o = a.Ob + (((size_t)branch * a.v.N + q.tok) * a.v.Hq + q.h) * D + 8 * h;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        bf16x8 w;
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = (__bf16)(st.o[db][8 * k + i] * inv);
        *reinterpret_cast<bf16x8 *>(o + 32 * db + 16 * k) = w;
      }
    if (h == 0) a.lse[((size_t)branch * a.v.N + q.tok) * a.v.Hq + q.h] = lse2 * LN2;
  }
  return lse2;
}

constexpr float SCORE_FIX = 134217728.0f;  // 2^27: a row's scores sum to h_s <= 16 < 2^5

static_assert(T32<64, true>::BYTES == tile_bytes(64) && T32<128, true>::BYTES == tile_bytes(128), "the LDS plans count whole tiles");
// Top-k of one token's score row Sr[0 .. nb) out of rows of s_max <= MOST; marks: scratch of the wavefront where rows are longer than
// TOPK_IN_REGISTERS; hist: as in topk_wave_bits, for rows up to CMP_ONE_BLOCKS.
template <int MOST>
__device__ inline void topk_slot(const uint32_t *Sr, int s_max, int nb, int T, int b0, int32_t *row, uint32_t *marks, uint32_t *hist) {
  if (s_max <= 64) topk_wave_bits<1>(Sr, nb, T, b0, row, hist);
  else if (s_max <= 128) topk_wave_bits<2>(Sr, nb, T, b0, row, hist);
  else if (s_max <= 256) topk_wave_bits<4>(Sr, nb, T, b0, row, hist);
  else if (s_max <= 512) topk_wave_bits<8>(Sr, nb, T, b0, row, hist);
  else if (MOST <= 1024 || s_max <= 1024) topk_wave_bits<16>(Sr, nb, T, b0, row, hist);
  else if constexpr (MOST > 1024) {
    if (s_max <= 2048) topk_wave_bits<32>(Sr, nb, T, b0, row, hist);
    else if (s_max <= TOPK_IN_REGISTERS) topk_wave_bits<64>(Sr, nb, T, b0, row, hist);
    else topk_wave_u32(Sr, nb, T, b0, row, marks);
  }
}

// Sums over the HS heads of a token of a tile of probabilities (query rows x keys: the lane holds rows t32_row(i) of one key): HS of
// 8 or 16 leaves each lane with 16 / HS of the key's tokens, fewer heads with both lanes' worth.
template <int HS> constexpr int token_sum_count() { return HS == 16 ? 1 : 16 / HS; }
template <int HS>
__device__ inline void token_sums(const f32x16 &c, float (&v)[token_sum_count<HS>()]) {
  if constexpr (HS >= 8) {  // groups of four heads: t[u] of lane h = rows 8*u + 4*h .. +3
    float t[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) t[u] = ((c[4 * u] + c[4 * u + 1]) + c[4 * u + 2]) + c[4 * u + 3];
    auto pair = [](float x, float y) {  // x's two lanes added in lane 0, y's in lane 1
      const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
      return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    };
    if constexpr (HS == 8) {
      v[0] = pair(t[0], t[1]);
      v[1] = pair(t[2], t[3]);
    } else {
      v[0] = pair(t[0], t[2]) + pair(t[1], t[3]);
    }
  } else {
#pragma unroll
    for (int u = 0; u < token_sum_count<HS>(); ++u) {
      v[u] = c[HS * u];
#pragma unroll
      for (int j = 1; j < HS; ++j) v[u] += c[HS * u + j];
    }
  }
}
// Token (of the wavefront's 32 rows) that sum u belongs to.
template <int HS>
__device__ inline int token_of_sum(int u) {
  const int h = threadIdx.x >> 5 & 1;
  return HS >= 8 ? 2 * u + h : (8 * (HS * u >> 2) + 4 * h + (HS * u & 3)) / HS;
}

// Neighbouring keys whose additions go to the same word of a score row, eight of them as one (integer sums: the row holds the same
// bits).  Keys 8*j .. +7 of a tile are the lanes that differ in bits 0, 1 and 3 (t32_order).  blk: the lane's selection block, which does
// not fall with the key, so eight keys are of one block if the first and the last are.
struct KeyGroups {
  bool same;   // the lane's eight keys are of one block
  bool adds;   // whether the lane adds: the first of eight, or any where they are of several blocks
  bool often;  // at least half of the groups are of one block (uniform)
  template <int CTRL>
  __device__ static inline uint32_t from(uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false); }
  static constexpr int QUAD_FIRST = 0x00, QUAD_LAST = 0xFF, XOR_1 = 0xB1, XOR_2 = 0x4E, XOR_8 = 0x128;
  __device__ inline explicit KeyGroups(int blk) {
    const uint32_t first = from<QUAD_FIRST>(blk), last = from<QUAD_LAST>(blk), first8 = from<XOR_8>(first), last8 = from<XOR_8>(last);
    same = threadIdx.x & 8 ? last == first8 : first == last8;
    adds = !same || (threadIdx.x & 11) == 0;
    often = __popcll(__ballot(same)) >= 32;
  }
  __device__ inline uint32_t sum(uint32_t x) const {
    uint32_t s = x + from<XOR_1>(x);
    s += from<XOR_2>(s);
    s += from<XOR_8>(s);
    return same ? s : x;
  }
};
// Heads per KV head up to which the groups are looked for.  A lane has 16 / heads additions per tile (at least two), of which those of 32
// keys of one block wait for each other; with 16 columns it was 16 keys.  16 columns / one by one / grouped, us of the compression branch: 95k
// tokens in 16^3 selection blocks, ungrouped heads of 32 785 / 1672 / 728, 4 heads of 32 1478 / 1878 / 1252, of 64 1892 / 2369 / 1745;
// sequences of 1024-token blocks, 64 pooled keys each, 4 heads of 64 716 / 1054 / 526; blocks of four or five pooled keys, where groups
// are rarely of one block, 62k tokens, 4 heads of 64 977 / 995 / 1040.  With 8 and 16 heads one by one is ahead of 16 columns everywhere.
constexpr int GROUP_HEADS = 4;

// Selection scores (eq. (6), the normaliser known) of one 32-key tile: kb its first key, key and blk this lane's key and its selection
// block.  Scores NOT transposed (query rows x keys), the heads of a token added in the lane (token_sums), and one integer LDS atomic
// adds the sum onto the score row of the token.  l16: -lse per row (log2 units); row0: first score row of the wavefront's 32 rows.
struct ScoreRows {
  uint32_t *S;          // [tokens][s_max]
  const int *tok_info;  // [3][tokens]: a token's first key, the one behind its last, the first selection block of its item
  int tokens, s_max, re, s0;
  bool one;             // all tokens are of one item, whose keys end at re and whose blocks start at s0
};
template <int D, int HS, class Operand>
__device__ inline void score_tile(const bf16x8 (&qop)[D / 16], Operand operand, const f32x16 &l16, float sl2, const ScoreRows &r, int row0, int kb, int key, int blk) {
  f32x16 c = splat16(0.f);
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) c = mfma32(qop[ks], operand(ks), c);
#pragma unroll
  for (int i = 0; i < 16; ++i) c[i] = fast_exp2(__builtin_fmaf(c[i], sl2, l16[i]));
  constexpr int NV = token_sum_count<HS>();
  float v[NV];
  token_sums<HS>(c, v);
  const bool whole = r.one && kb + 32 <= r.re;
  if constexpr (HS <= GROUP_HEADS) {
    const KeyGroups grp(blk);
    if (whole && grp.often) {
#pragma unroll
      for (int u = 0; u < NV; ++u) {
        const uint32_t x = grp.sum((uint32_t)(v[u] * SCORE_FIX));
        if (grp.adds) atomicAdd(&r.S[(row0 + token_of_sum<HS>(u)) * r.s_max + (blk - r.s0)], x);
      }
      return;
    }
  }
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    const int tok = row0 + token_of_sum<HS>(u);
    if (whole) atomicAdd(&r.S[tok * r.s_max + (blk - r.s0)], (uint32_t)(v[u] * SCORE_FIX));
    else if (key >= r.tok_info[tok] && key < r.tok_info[r.tokens + tok])
      atomicAdd(&r.S[tok * r.s_max + (blk - r.tok_info[2 * r.tokens + tok])], (uint32_t)(v[u] * SCORE_FIX));
  }
}

// The scores of 32 query rows per wavefront over the keys [rs, re): ST tiles per step through LDS, of which a wavefront takes every
// KS-th from number k0.
template <int D, int HS, int NTHR, int ST, int KS>
__device__ inline void score_walk(const MfmaView &v, const bf16_t *Kg, uint32_t stride, const bf16x8 (&qop)[D / 16], unsigned char *stage0, int rs, int k0,
                                  const f32x16 &l16, const ScoreRows &r, int row0, float sl2) {
  using T = T32<D, true>;
  const typename T::Lanes ln = T::lanes();
  const int n = t32_order(threadIdx.x & 31), last = v.Nc - 1;
  T32Src<ST> src;
  src.stride = stride;
#pragma unroll
  for (int t = 0; t < ST; ++t) src.row[t] = Kg + (size_t)(32 * t) * stride;
  t32_pipeline<D, ST, NTHR, 32 * ST>(src, stage0, rs, r.re, [&](lds_cptr kt, int kb0) {
    // the selection blocks of this lane's keys, requested before the matrix instructions
    int blk[ST / KS];
#pragma unroll
    for (int t = 0; t < ST / KS; ++t) blk[t] = v.cmp_slc[min(kb0 + 32 * (k0 + t * KS) + n, last)];
#pragma unroll
    for (int t = 0; t < ST / KS; ++t) {
      const int kb = kb0 + 32 * (k0 + t * KS);
      const lds_cptr tile = kt + (k0 + t * KS) * T::BYTES;
      score_tile<D, HS>(qop, [&](int ks) { return T::row(tile, ln, ks); }, l16, sl2, r, row0, kb, kb + n, blk[t]);
    }
  });
}

// Compression branch (eq. (4) first term over the mean-pooled keys of eq. (5)), then the selection scores of
// eq. (6) accumulated per selection block in LDS as fixed-point integers (integer adds commute, so the result
// does not depend on scheduling), then the top-k.  (cmp_form.h says where; elsewhere m_walk_fwd and m_cmp_scores.)
// Bound: matrix and vector issue over both walks, at a clock that falls to 1.8 - 1.9 GHz under them: per 32 x 32 scores at head_dim
// 64 the first walk takes 256 matrix cycles and about 280 of exponentials, multiply-adds, conversions and sums (a synthetic copy:
// 226 ns per SIMD), the second 128 and about 250; the kernel takes about 1.45 times that.  32 query columns per wavefront against
// 16: half the LDS operands per matrix cycle, half the staging and barriers per column.  Three wavefronts per SIMD (157 registers
// and LDS for three workgroups); two: 17 % slower.  At head_dim 128 two (233 registers); in two kernels
// 62k tokens and 662 blocks took 3400 us for 3130.  With the accumulators moved about once in two tiles, and 2 and 30 registers
// spilled (t32_pipeline), 62k tokens 1314 us for 1297 now, 153k, heads of 128, 8900 for 8640.  The sums of the first walk cost 5 % more in the order that keeps the selected
// sets what they were (SumInOrder).  62k tokens, 2247 pooled keys, 16 heads of 64: 1497 -> 1278 us (16 columns before); 65k tokens
// in three sequences 848 -> 767; 11k tokens 94 -> 79; 2k tokens, 32 heads of 32: 21 -> 16; 153k tokens, 3884 pooled keys, heads of
// 128: 11.4 -> 8.7 ms.
template <int D, int HS, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D <= 64 ? 3 : 2))) void m_cmp_fwd(FwdArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  using T = T32<D, true>;
  unsigned char *stage0 = smem;
  constexpr int TPW = 32 / HS, TW = NW * TPW;  // tokens per wavefront, per workgroup
  const int s_max = a.v.s_max;
  int *again = (int *)(stage0 + 4 * T::BYTES);
  float *lse_l = (float *)(again + 4);       // [32*NW] per query row
  int *tok_info = (int *)(lse_l + 32 * NW);  // [3][TW]
  uint32_t *S = (uint32_t *)(tok_info + 3 * TW);
  const int wid = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const TileMap tm = xcd_tile_map((a.v.N + TW - 1) / TW, a.v.Hkv);
  if (!tm.valid) return;
  const int g = tm.g, wg_pos0 = tm.tile * TW;
  bf16x8 qop[D / 16];
  load_col<D>(a.Q, a.v, query_col(a.v, wg_pos0, g), qop);
  // the items of the workgroup's tokens are a range (sorted by item), and so are their keys
  const int it0 = uniform(a.v.tok_item[wg_pos0]), it1 = uniform(a.v.tok_item[min(wg_pos0 + TW, a.v.N) - 1]);
  const int rs = uniform(a.v.cmp_batch[it0]), re = uniform(a.v.cmp_batch[it1 + 1]), s0 = uniform(a.v.slc_batch[it0]);
  const bool one = it0 == it1;
  if (threadIdx.x == 0) *again = 0;
  for (int t = threadIdx.x; t < TW; t += 64 * NW) {
    const int item = a.v.tok_item[min(wg_pos0 + t, a.v.N - 1)];
    tok_info[t] = a.v.cmp_batch[item];
    tok_info[TW + t] = a.v.cmp_batch[item + 1];
    tok_info[2 * TW + t] = a.v.slc_batch[item];
  }
  uint32_t *hist = a.cnt ? S + (size_t)TW * s_max : nullptr;  // [Ns] tokens of the workgroup that selected a block
  for (int i = threadIdx.x; i < TW * s_max + (hist ? a.v.Ns : 0); i += 64 * NW) S[i] = 0u;
  __syncthreads();
  const bf16_t *Kg = a.v.Kc + (size_t)g * D, *Vg = a.v.Vc + (size_t)g * D;
  const uint32_t stride = (uint32_t)(a.v.Hkv * D);
  const float sl2 = in_vgpr(a.v.sl2);
  T32State<D, SumInOrder> st;
  const bool have_ref = fwd_branch<D, NW>(st, lse_l, qop, T32Src<2>{{Kg, Vg}, stride}, stage0, again, rs, re, one, a.v.tok_item, a.v.cmp_batch, a.v, wg_pos0, sl2);
  const float lse2 = finish<D>(a, st, lse_l, have_ref, 0, query_col(a.v, wg_pos0, g));
  if (lane < 32) lse_l[wid * 32 + lane] = -lse2;
  __syncthreads();
  f32x16 l16;
#pragma unroll
  for (int i = 0; i < 16; ++i) l16[i] = lse_l[wid * 32 + t32_row(i)];
  const ScoreRows rows{S, tok_info, TW, s_max, re, s0, one};
  score_walk<D, HS, 64 * NW, 2, 1>(a.v, Kg, stride, qop, stage0, rs, 0, l16, rows, wid * TPW, sl2);  // (two tiles per step: half the barriers)
  // ---- top-k: each wavefront serves its own token slots, one after the other
  for (int tl = 0; tl < TPW; ++tl) {
    const int slot = wid * TPW + tl, pos = wg_pos0 + slot;
    if (pos >= a.v.N) break;
    const int tok = a.v.perm[pos], it = a.v.tok_item[pos];
    const int b0 = a.v.slc_batch[it], nb = a.v.slc_batch[it + 1] - b0;
    int32_t *row = a.idx + ((size_t)tok * a.v.Hkv + g) * a.v.T;
    topk_slot<CMP_ONE_BLOCKS>(S + (size_t)slot * s_max, s_max, nb, a.v.T, b0, row, nullptr, hist);
  }
  if (!hist) return;
  __syncthreads();
  for (int i = threadIdx.x; i < a.v.Ns; i += 64 * NW)
    if (hist[i]) atomicAdd(&a.cnt[((size_t)(wg_pos0 / POS_TILE) * a.v.Hkv + g) * a.v.Ns + i], hist[i]);
}

// Window branch: keys are the tokens of the query's own window.  16 columns per wavefront -> now: 62k tokens, 16 heads of 64: 145 -> 115
// us, 21k in three 64^3 shells 44 -> 33, 3k in sequences 21 -> 9, 24k in four shells, heads of 128: 80 -> 52.  64 query rows per
// workgroup: the walk of one whose tokens lie in several windows starts where the first of them does, so a later window's first tile,
// whose maximum is the reference, holds only some of 32 keys, and the largest weight is then seldom the exact 1 it is against its own
// score.  With 128 rows there are twice as many such workgroups: 2-norm error of the output against 64 bits, 21k tokens in three 64^3 shells,
// 2.7355e-3 for 2.7332e-3 (16 columns: 2.7335e-3), and the kernel takes 101 us at 62k tokens, but 17 at 3k.
// CMP: the compression branch alone, over the pooled keys of the query's item, where m_cmp_scores forms the selection scores.
template <int D, int NW, bool CMP>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 32 ? 4 : D == 64 ? 3 : 2))) void m_walk_fwd(FwdArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char *stage0 = smem;
  int *again = (int *)(stage0 + 4 * T32<D, true>::BYTES);
  float *refs = (float *)(again + 4);
  const int TW = 32 * NW / a.v.hs;
  const TileMap tm = xcd_tile_map((a.v.N + TW - 1) / TW, a.v.Hkv);
  if (!tm.valid) return;
  const int g = tm.g, wg_pos0 = tm.tile * TW;
  bf16x8 qop[D / 16];
  load_col<D>(a.Q, a.v, query_col(a.v, wg_pos0, g), qop);
  // the items (windows) of the workgroup's tokens are neighbours, and so are their keys
  const int32_t *of_pos = CMP ? a.v.tok_item : a.v.tok_win, *start = CMP ? a.v.cmp_batch : a.v.win_start;
  const int r0 = uniform(of_pos[wg_pos0]), r1 = uniform(of_pos[min(wg_pos0 + TW, a.v.N) - 1]);
  const int rs = uniform(start[r0]), re = uniform(start[r1 + 1]);
  if (threadIdx.x == 0) *again = 0;
  __syncthreads();
  T32State<D, std::conditional_t<CMP, SumInOrder, SumParts>> st;
  const T32Src<2> src{{(CMP ? a.v.Kc : a.v.Ks) + (size_t)g * D, (CMP ? a.v.Vc : a.v.Vs) + (size_t)g * D}, (uint32_t)(a.v.Hkv * D)};
  const bool have_ref = fwd_branch<D, NW>(st, refs, qop, src, stage0, again, rs, re, r0 == r1, of_pos, start, a.v, wg_pos0, in_vgpr(a.v.sl2));
  const QCol q = query_col(a.v, wg_pos0, g);
  const float lse2 = finish<D>(a, st, refs, have_ref, CMP ? 0 : 2, q);
  if (CMP && q.valid) a.nlse[(size_t)q.pos * a.v.Hq + q.h] = -lse2;  // (both lanes of a column: the same)
}

// Selection scores of eq. (6) and top-k behind m_walk_fwd<.., true>: CW * KS wavefronts share the score rows of 32 * CW query rows, and
// KS of them the 32 rows of a group, of which each takes every KS-th tile of 32 pooled keys.  The scores are the same products and
// integer additions as in m_cmp_fwd, so the selected sets are too.  ST tiles per step go through LDS, or (ST = 0, CW = 1) every
// wavefront loads the rows of its tiles itself, the next tile's in flight: no tile is wanted twice, and LDS is left to the score rows.
// Bound: with the tiles in LDS the sum of matrix and vector issue; without, the L1 cache (4 KB of key rows at head_dim 64 for 128 matrix
// cycles).
template <int D, int HS, int CW, int KS, int ST>
__global__ __launch_bounds__(64 * CW * KS) __attribute__((amdgpu_waves_per_eu(D <= 64 ? 4 : HS == 1 ? 2 : 3))) void m_cmp_scores(FwdArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  using T = T32<D, true>;
  constexpr int NW = CW * KS, TPW = 32 / HS, TW = CW * TPW;
  static_assert(ST > 0 ? ST % KS == 0 : CW == 1, "a tile loaded by one wavefront is used by one");
  const int s_max = a.v.s_max, N = a.v.N;
  int *tok_info = (int *)(smem + 2 * ST * T::BYTES);  // [3][TW]
  uint32_t *S = (uint32_t *)(tok_info + 3 * TW);      // [TW][s_max]
  const int wid = uniform(threadIdx.x >> 6), n = threadIdx.x & 31, h = threadIdx.x >> 5 & 1, group = wid % CW, k0 = wid / CW;
  const TileMap tm = xcd_tile_map((N + TW - 1) / TW, a.v.Hkv);
  if (!tm.valid) return;
  const int g = tm.g, wg_pos0 = tm.tile * TW, pos0 = wg_pos0 + group * TPW;
  bf16x8 qop[D / 16];
  const bf16_t *src = a.Q + ((size_t)a.v.perm[min(pos0 + n / HS, N - 1)] * a.v.Hq + g * HS + n % HS) * D + 8 * h;
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) qop[ks] = ld8(src + 16 * ks);
  f32x16 l16;
#pragma unroll
  for (int i = 0; i < 16; ++i) l16[i] = a.nlse[(size_t)min(pos0 + t32_row(i) / HS, N - 1) * a.v.Hq + g * HS + t32_row(i) % HS];
  const int it0 = uniform(a.v.tok_item[wg_pos0]), it1 = uniform(a.v.tok_item[min(wg_pos0 + TW, N) - 1]);
  const int rs = uniform(a.v.cmp_batch[it0]), re = uniform(a.v.cmp_batch[it1 + 1]), s0 = uniform(a.v.slc_batch[it0]);
  if (threadIdx.x < TW) {
    const int item = a.v.tok_item[min(wg_pos0 + (int)threadIdx.x, N - 1)];
    tok_info[threadIdx.x] = a.v.cmp_batch[item];
    tok_info[TW + threadIdx.x] = a.v.cmp_batch[item + 1];
    tok_info[2 * TW + threadIdx.x] = a.v.slc_batch[item];
  }
  for (int i = threadIdx.x; i < TW * s_max; i += 64 * NW) S[i] = 0u;
  __syncthreads();
  const uint32_t stride = (uint32_t)(a.v.Hkv * D);
  const bf16_t *Kg = a.v.Kc + (size_t)g * D;
  const float sl2 = in_vgpr(a.v.sl2);
  const ScoreRows rows{S, tok_info, TW, s_max, re, s0, it0 == it1};
  if constexpr (ST > 0) {
    score_walk<D, HS, 64 * NW, ST, KS>(a.v, Kg, stride, qop, smem, rs, k0, l16, rows, group * TPW, sl2);
  } else {
    struct Keys { bf16x8 op[D / 16]; int blk; } ka, kb;
    constexpr int STEP = 32 * NW;
    auto load = [&](int key, Keys &k) {  // the tile at key, or (past the end: not used) the first one; rows past the last key are padding
      const int row = (key < re ? key : rs) + n;
      const bf16_t *x = Kg + ((uint32_t)row * stride + (uint32_t)(8 * h));
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks) k.op[ks] = ld8(x + 16 * ks);
      k.blk = a.v.cmp_slc[min(row, a.v.Nc - 1)];
    };
    auto tile = [&](int key, const Keys &k) {
      score_tile<D, HS>(qop, [&](int ks) { return k.op[ks]; }, l16, sl2, rows, 0, key, key + n, k.blk);
    };
    load(rs + 32 * wid, ka);
    for (int key = rs + 32 * wid; key < re; key += 2 * STEP) {
      load(key + STEP, kb);
      tile(key, ka);
      if (key + STEP >= re) break;
      load(key + 2 * STEP, ka);
      tile(key + STEP, kb);
    }
    __syncthreads();
  }
  for (int slot = wid; slot < TW && wg_pos0 + slot < N; slot += NW) {
    const int pos = wg_pos0 + slot, tok = a.v.perm[pos], it = a.v.tok_item[pos];
    const int b0 = a.v.slc_batch[it], nb = a.v.slc_batch[it + 1] - b0;
    topk_slot<INT_MAX>(S + (size_t)slot * s_max, s_max, nb, a.v.T, b0, a.idx + ((size_t)tok * a.v.Hkv + g) * a.v.T,
                       S + (size_t)TW * s_max + (size_t)wid * ((s_max + 31) >> 5), nullptr);
  }
}
// (raises the dynamic LDS limit once per process for every instantiation)
template <class Kernel>
void allow_lds(std::once_flag &once, Kernel kernel) {
  std::call_once(once, [&] { (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_CU); });
}

template <int D, int HS, int CW, int KS, int ST>
void launch_scores(const FwdArgs &a, hipStream_t s) {
  static std::once_flag once;
  allow_lds(once, m_cmp_scores<D, HS, CW, KS, ST>);
  constexpr int TW = CW * 32 / HS;
  m_cmp_scores<D, HS, CW, KS, ST><<<dim3(xcd_grid_size((a.v.N + TW - 1) / TW, a.v.Hkv)), 64 * CW * KS, scores_lds_bytes(D, HS, CW, CW * KS, ST, a.v.s_max), s>>>(a);
}
template <int D, int HS>
void launch_scores(const FwdArgs &a, CmpForm form, hipStream_t s) {
  if constexpr (HS > 1)
    if (form == CmpForm::tiles_in_lds) return launch_scores<D, HS, 2, 2, 2>(a, s);
  if (form == CmpForm::own_tiles_4) launch_scores<D, HS, 1, 4, 0>(a, s);
  else launch_scores<D, HS, 1, 8, 0>(a, s);
}

template <int D, int NW, bool CMP>
void launch_walk(const FwdArgs &a, hipStream_t s) {
  const int tw = 32 * NW / a.v.hs;
  m_walk_fwd<D, NW, CMP><<<dim3(xcd_grid_size((a.v.N + tw - 1) / tw, a.v.Hkv)), 64 * NW, 4 * T32<D, true>::BYTES + 16 + 32 * NW * 4, s>>>(a);
}

// Whether the window branch takes 128 query rows per workgroup instead of 64: windows of 500 tokens on average.  There the error is the
// same with both (1000 tokens, ungrouped heads, one workgroup of 128 rows in eight over two windows: output 2.32692e-3 for 2.32694e-3,
// lse 1.2220e-5 for 1.2225e-5; 512: 1.81689e-5 both), and the larger ones stage half as often.  64 / 128 rows, us: 65k tokens in windows of 512
// 229 / 202 (16 columns: 272), 4096 1617 / 1405 (1767), 40k in one 9488 / 8220 (10480); ungrouped 8k in one 160 / 133 (137); 3k in 512 18.9 / 19.1.
inline bool windows_long(const MfmaView &v) { return v.N >= 500LL * v.Nw; }

template <int D, int HS>
void launch_cmp(const FwdArgs &a, hipStream_t s) {
  constexpr int NW = 4;
  const CmpForm form = cmp_form(D, HS, a.v.s_max);
  if constexpr (HS >= 4)
    if (form == CmpForm::one_kernel) {
      static std::once_flag once;
      allow_lds(once, m_cmp_fwd<D, HS, NW>);
      constexpr int TW = 32 * NW / HS;
      m_cmp_fwd<D, HS, NW><<<dim3(xcd_grid_size((a.v.N + TW - 1) / TW, a.v.Hkv)), 64 * NW,
                                cmp_lds_bytes(D, NW, HS, a.v.s_max) + (a.cnt ? (size_t)a.v.Ns * 4 : 0), s>>>(a);
      return;
    }
  launch_walk<D, NW, true>(a, s);
  launch_scores<D, HS>(a, form, s);
}
template <int D>
void launch_cmp(const FwdArgs &a, hipStream_t s) {
  switch (a.v.hs) {
    case 1: return launch_cmp<D, 1>(a, s);
    case 2: return launch_cmp<D, 2>(a, s);
    case 4: return launch_cmp<D, 4>(a, s);
    case 8: return launch_cmp<D, 8>(a, s);
    default: return launch_cmp<D, 16>(a, s);
  }
}

template <int D>
int launch_forward(FwdArgs a, const bf16_t *gates, bf16_t *out, SlcKeep keep, const SelIndex &sel, const SlcPartials &part, hipStream_t s) {
  {
    ProfScope ps(PROF_CMP_FWD, s);
    launch_cmp<D>(a, s);
  }
  {
    ProfScope ps(PROF_FWD_INVERT, s);
    const int rc = sel_index_build(a.idx, a.v.perm, a.v.slc_start, a.v.N, a.v.Hkv, a.v.T, a.v.Ns, sel, true, true, false, a.cnt != nullptr, s);
    if (rc != SSA_OK) return rc;
  }
  {
    ProfScope ps(PROF_SLC_FWD, s);
    const int rc = slc_forward_kernel(a.v, D, a.Q, sel, part, s);
    if (rc != SSA_OK) return rc;
  }
  {
    ProfScope ps(PROF_WIN_FWD, s);
    if (windows_long(a.v)) launch_walk<D, 4, false>(a, s);
    else launch_walk<D, 2, false>(a, s);
  }
  {
    ProfScope ps(PROF_COMBINE, s);
    const int rc = slc_merge_kernel(a.v, D, part, a.idx, gates, a.Ob, a.lse, out, keep, s);
    if (rc != SSA_OK) return rc;
  }
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}

}  // namespace

int mfma_forward_kernels(const MfmaView &v, int D, const void *q, const void *gates, void *out, float *lse,
                         int32_t *idx, void *out_branch, SlcKeep keep, const SelIndex &sel, const SlcPartials &part,
                         hipStream_t s) {
  const bool counts = sel_counted(D, v.hs, v.s_max, v.N, v.Hkv, v.Ns);
  FwdArgs a{v, (const bf16_t *)q, (bf16_t *)out_branch, lse, idx, part.ml, counts ? sel.cnt : nullptr};
  switch (D) {
    case 32: return launch_forward<32>(a, (const bf16_t *)gates, (bf16_t *)out, keep, sel, part, s);
    case 64: return launch_forward<64>(a, (const bf16_t *)gates, (bf16_t *)out, keep, sel, part, s);
    case 128: return launch_forward<128>(a, (const bf16_t *)gates, (bf16_t *)out, keep, sel, part, s);
    default: return SSA_ERR_UNSUPPORTED;
  }
}
