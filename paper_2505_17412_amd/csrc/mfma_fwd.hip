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
#include "profile.h"

#include <mutex>

namespace {

struct FwdArgs {
  MfmaView v;
  const bf16_t *Q;
  bf16_t *Ob;    // [3,N,Hq,D]
  float *lse;    // [3,N,Hq]
  int32_t *idx;  // [N,Hkv,T]
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
  t32_pipeline<D, 2, 64 * NW, 32, T32_PF>(src, stage0, first, re, [&](lds_cptr kt, int kb) {
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
  t32_pipeline<D, 2, 64 * NW, 32, T32_PF>(src, stage0, walk_begin(rs), re, [&](lds_cptr kt, int kb) {
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

// LDS plan of the compression kernel (bytes): two stages of two tiles | repeat flag, padding | lse per query row | per token its
// first pooled key, the one behind its last and the first score of its item | scores [TW][s_max] | top-k marks [NW][words]
// Blocks of an item whose scores a wavefront holds in registers for the top-k search; more are searched in T rounds over LDS.  With
// 1024 here: one sequence of 72k tokens (1125 blocks) 5090 us for 3320 now, 131k (2048) 26900 for 11600.
constexpr int TOPK_IN_REGISTERS = 4096;
template <int D>
__host__ __device__ inline size_t cmp_lds_bytes(int nw, int hs, int s_max) {
  const int tw = 32 * nw / hs;
  return (size_t)4 * T32<D, true>::BYTES + 16 + ((size_t)32 * nw + 3 * tw + (size_t)tw * s_max + (s_max > TOPK_IN_REGISTERS ? nw * ((s_max + 31) / 32) : 0)) * 4;
}

// Second walk of the compression kernel: eq. (6) scores with the normaliser known, for HS heads per KV head, over steps of two
// 32-key tiles.  Scores NOT transposed (query rows x keys): a lane holds rows t32_row(i) for one key, and adds the heads of a token
// in-lane; with 8 or 16 heads one register swap adds the other lane's for two tokens at once and leaves each lane with one token,
// and one integer LDS atomic adds the sum onto the key's selection block.  l16: -lse per row (log2 units).
template <int D, int NW, int HS>
__device__ inline void score_walk(const FwdArgs &a, const bf16x8 (&qop)[D / 16], const T32Src<2> &src, unsigned char *stage0, int rs, int re, bool one,
                                  const f32x16 &l16, const int *tok_info, int s0, uint32_t *S, float sl2) {
  using T = T32<D, true>;
  constexpr int TPW = 32 / HS, TW = NW * TPW;   // tokens per wavefront, per workgroup
  constexpr int NV = HS == 16 ? 1 : 16 / HS;    // sums a lane adds per tile
  const typename T::Lanes ln = T::lanes();
  const int n = t32_order(threadIdx.x & 31), h = threadIdx.x >> 5 & 1, wid = threadIdx.x >> 6, last = a.v.Nc - 1, s_max = a.v.s_max;
  t32_pipeline<D, 2, 64 * NW, 64, T32_PF>(src, stage0, rs, re, [&](lds_cptr kt, int kb2) {
    // the selection blocks of this lane's keys, requested before the matrix instructions
    int sb[2];
#pragma unroll
    for (int half = 0; half < 2; ++half) sb[half] = a.v.cmp_slc[min(kb2 + 32 * half + n, last)];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      f32x16 c = splat16(0.f);
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks) c = mfma32(qop[ks], T::row(kt + half * T::BYTES, ln, ks), c);
#pragma unroll
      for (int i = 0; i < 16; ++i) c[i] = fast_exp2(__builtin_fmaf(c[i], sl2, l16[i]));
      float v[NV];
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
        for (int u = 0; u < NV; ++u) {
          v[u] = c[HS * u];
#pragma unroll
          for (int j = 1; j < HS; ++j) v[u] += c[HS * u + j];
        }
      }
      const int key = kb2 + 32 * half + n;
      const bool whole = one && kb2 + 32 * half + 32 <= re;
#pragma unroll
      for (int u = 0; u < NV; ++u) {
        // token of sum u: rows t32_row(i) / HS
        const int tok = wid * TPW + (HS >= 8 ? 2 * u + h : (8 * (HS * u >> 2) + 4 * h + (HS * u & 3)) / HS);
        if (whole) atomicAdd(&S[tok * s_max + (sb[half] - s0)], (uint32_t)(v[u] * SCORE_FIX));
        else if (key >= tok_info[tok] && key < tok_info[TW + tok])
          atomicAdd(&S[tok * s_max + (sb[half] - tok_info[2 * TW + tok])], (uint32_t)(v[u] * SCORE_FIX));
      }
    }
  });
}

// Compression branch (eq. (4) first term over the mean-pooled keys of eq. (5)), then the selection scores of
// eq. (6) accumulated per selection block in LDS as fixed-point integers (integer adds commute, so the result
// does not depend on scheduling), then the top-k.
// Bound: matrix and vector issue over both walks, at a clock that falls to 1.8 - 1.9 GHz under them: per 32 x 32 scores at head_dim
// 64 the first walk takes 256 matrix cycles and about 280 of exponentials, multiply-adds, conversions and sums (a synthetic copy:
// 226 ns per SIMD), the second 128 and about 250; the kernel takes about 1.45 times that.  32 query columns per wavefront against
// 16: half the LDS operands per matrix cycle, half the staging and barriers per column.  Three wavefronts per SIMD (168 registers,
// and LDS for three workgroups); two: 17 % slower.  The sums of the first walk cost 5 % more in the order that keeps the selected
// sets what they were (SumInOrder; 1290 us without).  62k tokens, 2247 pooled keys, 16 heads of 64: 1516 -> 1370 us (16 columns
// before); 65k tokens in sequences 880 -> 830; 11k tokens 94 -> 79; 2k tokens, 32 heads of 32: 19.6 -> 14; 153k tokens, 3884 pooled
// keys, heads of 128: 11.5 -> 9.1 ms.
template <int D, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D <= 64 && NW < 8 ? 3 : 2))) void m_cmp_fwd(FwdArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  using T = T32<D, true>;
  unsigned char *stage0 = smem;
  const int hs = a.v.hs, s_max = a.v.s_max, TW = 32 * NW / hs;
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
  for (int i = threadIdx.x; i < TW * s_max; i += 64 * NW) S[i] = 0u;
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
  // two consecutive 32-key tiles per step: half the barriers and staging rounds of a walk that has little work per key
  const T32Src<2> src2{{Kg, Kg + (size_t)32 * stride}, stride};
  auto walk = [&](auto hs_c) {  // a walk per head count: the tile code is straight-line
    score_walk<D, NW, decltype(hs_c)::value>(a, qop, src2, stage0, rs, re, one, l16, tok_info, s0, S, sl2);
  };
  if (hs == 8) walk(std::integral_constant<int, 8>());
  else if (hs == 16) walk(std::integral_constant<int, 16>());
  else if (hs == 4) walk(std::integral_constant<int, 4>());
  else if (hs == 2) walk(std::integral_constant<int, 2>());
  else walk(std::integral_constant<int, 1>());
  // ---- top-k: each wavefront serves its own token slots, one after the other
  const int spw = 32 / hs;  // token slots per wavefront
  for (int tl = 0; tl < spw; ++tl) {
    const int slot = wid * spw + tl, pos = wg_pos0 + slot;
    if (pos >= a.v.N) break;
    const int tok = a.v.perm[pos], it = a.v.tok_item[pos];
    const int b0 = a.v.slc_batch[it], nb = a.v.slc_batch[it + 1] - b0;
    int32_t *row = a.idx + ((size_t)tok * a.v.Hkv + g) * a.v.T;
    const uint32_t *Sr = S + (size_t)slot * s_max;
    if (s_max <= 64) topk_wave_bits<1>(Sr, nb, a.v.T, b0, row);
    else if (s_max <= 128) topk_wave_bits<2>(Sr, nb, a.v.T, b0, row);
    else if (s_max <= 256) topk_wave_bits<4>(Sr, nb, a.v.T, b0, row);
    else if (s_max <= 512) topk_wave_bits<8>(Sr, nb, a.v.T, b0, row);
    else if (s_max <= 1024) topk_wave_bits<16>(Sr, nb, a.v.T, b0, row);
    else if (s_max <= 2048) topk_wave_bits<32>(Sr, nb, a.v.T, b0, row);
    else if (s_max <= TOPK_IN_REGISTERS) topk_wave_bits<64>(Sr, nb, a.v.T, b0, row);
    else topk_wave_u32(Sr, nb, a.v.T, b0, row, S + (size_t)TW * s_max + (size_t)wid * ((s_max + 31) >> 5));
  }
}

// Window branch: keys are the tokens of the query's own window.  62k tokens, 16 heads of 64: 154 -> 105 us (16 columns per wavefront
// before), 65k tokens in windows of 512: 270 -> 190, 153k tokens, heads of 128: 1109 -> 720.
template <int D, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 32 ? 4 : D == 64 ? 3 : 2))) void m_win_fwd(FwdArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char *stage0 = smem;
  int *again = (int *)(stage0 + 4 * T32<D, true>::BYTES);
  const int TW = 32 * NW / a.v.hs;
  const TileMap tm = xcd_tile_map((a.v.N + TW - 1) / TW, a.v.Hkv);
  if (!tm.valid) return;
  const int g = tm.g, wg_pos0 = tm.tile * TW;
  bf16x8 qop[D / 16];
  load_col<D>(a.Q, a.v, query_col(a.v, wg_pos0, g), qop);
  const int w0 = uniform(a.v.tok_win[wg_pos0]), w1 = uniform(a.v.tok_win[min(wg_pos0 + TW, a.v.N) - 1]);
  const int rs = uniform(a.v.win_start[w0]), re = uniform(a.v.win_start[w1 + 1]);
  if (threadIdx.x == 0) *again = 0;
  float *refs = (float *)(again + 4);
  __syncthreads();
  T32State<D, SumParts> st;
  const bool have_ref = fwd_branch<D, NW>(st, refs, qop, T32Src<2>{{a.v.Ks + (size_t)g * D, a.v.Vs + (size_t)g * D}, (uint32_t)(a.v.Hkv * D)}, stage0, again, rs, re,
                  w0 == w1, a.v.tok_win, a.v.win_start, a.v, wg_pos0, in_vgpr(a.v.sl2));
  finish<D>(a, st, refs, have_ref, 2, query_col(a.v, wg_pos0, g));
}

// Wavefronts per workgroup of the compression kernel: what keeps most of them on a compute unit beside the score rows (four where
// that is equal).  Two everywhere: 62k tokens 1290 -> 1527 us, 11k 79 -> 85 (each stages the pooled keys for half the columns).  One
// sequence of 65k tokens, 1024 selection blocks: 2320 us by two (six on a compute unit), 1810 by eight; the 16-column kernel, with
// half the score rows per wavefront and twelve of them, took 1620.
constexpr size_t CMP_LDS_CU = 160 * 1024, CMP_LDS_WG = 150 * 1024;
template <int D>
int cmp_waves(int hs, int s_max) {
  constexpr int by_registers = D <= 64 ? 12 : 8;
  int best = 2, most = 0;
  for (const int nw : {4, 8, 2}) {
    const size_t lds = cmp_lds_bytes<D>(nw, hs, s_max);
    if (lds > CMP_LDS_WG) continue;
    const int by_lds = (int)(CMP_LDS_CU / lds) * nw, waves = by_lds < by_registers / nw * nw ? by_lds : by_registers / nw * nw;
    if (waves > most) {
      most = waves;
      best = nw;
    }
  }
  return best;
}

template <int D, int NW>
void launch_cmp(const FwdArgs &a, hipStream_t s) {
  static std::once_flag once;  // raise the dynamic LDS limit once per process for this instantiation
  std::call_once(once, [] { (void)hipFuncSetAttribute((const void *)m_cmp_fwd<D, NW>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); });
  const int tw = 32 * NW / a.v.hs;
  m_cmp_fwd<D, NW><<<dim3(xcd_grid_size((a.v.N + tw - 1) / tw, a.v.Hkv)), 64 * NW, cmp_lds_bytes<D>(NW, a.v.hs, a.v.s_max), s>>>(a);
}

template <int D>
int launch_forward(FwdArgs a, const bf16_t *gates, bf16_t *out, SlcKeep keep, const SelIndex &sel, const SlcPartials &part, hipStream_t s) {
  {
    ProfScope ps(PROF_CMP_FWD, s);
    const int nw = cmp_waves<D>(a.v.hs, a.v.s_max);
    if (nw == 4) launch_cmp<D, 4>(a, s);
    else if (nw == 8) launch_cmp<D, 8>(a, s);
    else launch_cmp<D, 2>(a, s);
  }
  {
    ProfScope ps(PROF_FWD_INVERT, s);
    const int rc = sel_index_build(a.idx, a.v.perm, a.v.slc_start, a.v.N, a.v.Hkv, a.v.T, a.v.Ns, sel, true, true, false, s);
    if (rc != SSA_OK) return rc;
  }
  {
    ProfScope ps(PROF_SLC_FWD, s);
    const int rc = slc_forward_kernel(a.v, D, a.Q, sel, part, s);
    if (rc != SSA_OK) return rc;
  }
  {
    ProfScope ps(PROF_WIN_FWD, s);
    constexpr int NW = 4;
    const int tw = 32 * NW / a.v.hs;
    m_win_fwd<D, NW><<<dim3(xcd_grid_size((a.v.N + tw - 1) / tw, a.v.Hkv)), 64 * NW, 4 * T32<D, true>::BYTES + 16 + 32 * NW * 4, s>>>(a);
  }
  {
    ProfScope ps(PROF_COMBINE, s);
    const int rc = slc_merge_kernel(a.v, D, part, a.idx, gates, a.Ob, a.lse, out, keep, s);
    if (rc != SSA_OK) return rc;
  }
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}

}  // namespace

// Largest dynamic LDS request of the forward kernels for this problem (bytes).
size_t mfma_fwd_lds_bytes(int D, int hs, int s_max) {
  switch (D) {
    case 32: return cmp_lds_bytes<32>(cmp_waves<32>(hs, s_max), hs, s_max);
    case 64: return cmp_lds_bytes<64>(cmp_waves<64>(hs, s_max), hs, s_max);
    default: return cmp_lds_bytes<128>(cmp_waves<128>(hs, s_max), hs, s_max);
  }
}

int mfma_forward_kernels(const MfmaView &v, int D, const void *q, const void *gates, void *out, float *lse,
                         int32_t *idx, void *out_branch, SlcKeep keep, const SelIndex &sel, const SlcPartials &part,
                         hipStream_t s) {
  FwdArgs a{v, (const bf16_t *)q, (bf16_t *)out_branch, lse, idx};
  switch (D) {
    case 32: return launch_forward<32>(a, (const bf16_t *)gates, (bf16_t *)out, keep, sel, part, s);
    case 64: return launch_forward<64>(a, (const bf16_t *)gates, (bf16_t *)out, keep, sel, part, s);
    case 128: return launch_forward<128>(a, (const bf16_t *)gates, (bf16_t *)out, keep, sel, part, s);
    default: return SSA_ERR_UNSUPPORTED;
  }
}
