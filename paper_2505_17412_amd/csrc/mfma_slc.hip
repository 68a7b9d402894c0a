// Selection branch of SSA on bf16 MFMA for gfx950, block-centric: Algorithm 1 with its two loops exchanged, forward and
// dQ, and the kernels that merge the per-block partial results (the forward one also forms the gated sum of eq. (4)).
// A translation unit of its own: these kernels have no barrier in their inner loops and long straight-line tile code,
// and are compiled with an instruction scheduler setting of their own (see build.py).
#include "mfma_common.h"
#include "mfma_launch.h"
#include "mfma_qc.h"
#include "mfma_t32.h"

#include <mutex>

namespace {

// ---------------------------------------------------------------------------------------------------------
// Selection branch, block-centric (Algorithm 1 with the loops exchanged): the outer loop runs over the selected blocks,
// the inner one over the query tokens that selected the block.  A workgroup takes one (KV head, selection block) and a
// chunk of up to BC_CHUNK tokens of that block's selector list, puts the block's K and V rows into LDS ONCE (up to KSEG
// keys; longer blocks in several segments) and lets every wavefront run, on its own and without any barrier, through
// steps of 32/h_s tokens: all 32 query columns of a matrix tile then take part in every key tile (nothing is
// computed for a token that did not select the block) and no wavefront waits for another.  The price is one partial result per
// (token, KV head, selected block): the unnormalised output in bf16 with its reference exponent and sum (Algorithm 1's o, m, l for
// that block alone), merged per token afterwards (m_slc_merge).  A wavefront that meets a block longer than KSEG picks its own
// partial up again for the next segment.
// Bound: for blocks of ordinary length the sum of matrix and vector issue (a tile of 32 x 32 scores at head_dim 64 is 288 matrix
// cycles and about 250 of exponentials, conversions and multiply-adds; a synthetic copy takes 226 ns per SIMD at four wavefronts,
// with the clock down to 1.8 GHz), beside the partial rows going out (2.0 GB at 62k tokens = 440 us of writing; without any tile
// but the last of a block 770 us).  32 columns per wavefront against 16: an operand read from LDS feeds twice the matrix work, and
// the four SIMDs no longer ask LDS for every cycle it has.  Four wavefronts per SIMD at head_dim 64 (126 registers; the query rows of
// the next step are loaded into the registers of this step's as soon as its last scores are formed).  A step's stores are not waited
// for by the next one (t32_store_rows, wait_loads).  62k tokens, 16 heads of 64, top-16: 989 -> 874 us; 11k tokens, top-8: 154 ->
// 114; sequences of 64-key blocks 736 -> 612; 153k tokens, heads of 128: 10.2 -> 9.2 ms (with 16 columns per wavefront before).
// ---------------------------------------------------------------------------------------------------------
struct BcFwdArgs {
  MfmaView v;
  const bf16_t *Q;
  const int32_t *sel_list, *chunk_start;  // lists of caller indices
  const uint8_t *sel_rank;
  const ChunkRef *chunk_order;
  bf16_t *po;  // [N][Hkv][T][hs][D] and a spare row
  float *pml;  // [N][Hkv][T][hs][2], the same
};

// LDS plan (bytes): K tiles | V tiles (KSEG/32 tiles each) | chunk entries [BC_CHUNK][2] | what the last tile's scores start from
template <int D, int KSEG>
constexpr size_t bc_lds_bytes() { return (size_t)2 * (KSEG / 32) * T32<D, false>::BYTES + (size_t)2 * BC_CHUNK * sizeof(int) + 32 * sizeof(float); }

// Query operands and partial-row index of one wavefront step: column n stands for chunk entry step*(32/h_s) + n/h_s, head
// n % h_s of the KV group.  Columns past the end of the chunk take the query rows of its last entry and the spare partial row.
template <int D>
struct BcRows {
  bf16x8 qop[D / 16];
  uint32_t prow;  // ((tok*Hkv + g)*T + rank)*hs + head: row of the partial arrays (below 2^32: N*Hq*T is), or the spare one
};

// ent: per chunk entry the byte offset of the token's query rows of this KV group and its first partial row.
template <int D>
__device__ inline void bc_load_rows(const unsigned char *Q, const uint2 *ent, int step, int cnt, int lg_tpw, int slot, uint32_t lane_off,
                                    int hl, uint32_t spare, BcRows<D> &r) {
  const int e = (step << lg_tpw) + slot;
  const uint2 x = ent[min(e, cnt - 1)];
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) r.qop[ks] = *reinterpret_cast<const bf16x8 *>(Q + (x.x + lane_off) + 32 * ks);
  r.prow = e < cnt ? x.y + hl : spare;
}

// The 8 + 8 dims of block db that a lane holds of its column's row.
template <int D>
__device__ inline void bc_pick_up_row(const bf16_t *rows, uint32_t prow, f32x16 (&o)[D / 32]) {
  const bf16_t *src = rows + (size_t)prow * D + 8 * (threadIdx.x >> 5 & 1);
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const bf16x8 x = ld8(src + 32 * db + 16 * k);
#pragma unroll
      for (int i = 0; i < 8; ++i) o[db][8 * k + i] = (float)x[i];
    }
}

// The partial of the earlier segments, picked up again.  Columns past the end of the chunk start from nothing: the spare row holds
// whatever column of whatever workgroup wrote it last.
template <int D>
__device__ inline void bc_pick_up(const BcFwdArgs &a, uint32_t prow, uint32_t spare, T32State<D, SumParts> &st) {
  if (prow == spare) {
    t32_clear(st);
    st.m = 0.f;
    return;
  }
  const float2 ml = *reinterpret_cast<const float2 *>(a.pml + (size_t)prow * 2);
  st.m = ml.x;
  st.l.part[0] = threadIdx.x & 32 ? 0.f : ml.y;
  st.l.part[1] = 0.f;
  bc_pick_up_row<D>(a.po, prow, st.o);
}

template <int D, int NW, int KSEG, int WPE>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(WPE))) void m_slc_fwd_bc(BcFwdArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  using T = T32<D, false>;
  constexpr int MAXT = KSEG / 32;
  unsigned char *Kt = smem, *Vt = Kt + MAXT * T::BYTES;
  uint2 *ent = (uint2 *)(Vt + MAXT * T::BYTES);
  float *tail = (float *)(ent + BC_CHUNK);
  const int wid = uniform(threadIdx.x >> 6), h = threadIdx.x >> 5 & 1, n = threadIdx.x & 31;
  const int hs = a.v.hs, Hkv = a.v.Hkv, Ns = a.v.Ns;
  const int wi = blockIdx.x;
  if (wi >= a.chunk_start[Hkv * Ns]) return;
  const ChunkRef cr = a.chunk_order[wi];
  const int key = uniform(cr.key), g = key / Ns, blk = key % Ns;
  const int kbeg = uniform(a.v.slc_start[blk]), kend = uniform(a.v.slc_start[blk + 1]);
  const int qbeg = uniform(cr.first), cnt = uniform(cr.count);
  for (int i = threadIdx.x; i < cnt; i += 64 * NW) {
    const uint32_t tok = (uint32_t)a.sel_list[qbeg + i];
    ent[i] = make_uint2((tok * a.v.Hq + g * hs) * (D * 2), ((tok * Hkv + g) * a.v.T + a.sel_rank[qbeg + i]) * hs);
  }
  const int lg_tpw = 31 - __builtin_clz(32 / hs), slot = n / hs, hl = n % hs;
  const uint32_t lane_off = (uint32_t)(hl * D * 2 + 16 * h);
  const unsigned char *Qb = (const unsigned char *)a.Q;
  const int n_it = (cnt + (1 << lg_tpw) - 1) >> lg_tpw;
  const uint32_t kstride = (uint32_t)(Hkv * D);
  const float sl2 = in_vgpr(a.v.sl2);
  const typename T::Lanes ln = T::lanes();
  const lds_cptr kl = (lds_cptr)Kt, vl = (lds_cptr)Vt;
  const uint32_t spare = (uint32_t)((size_t)a.v.N * a.v.Hq * a.v.T);  // behind the last partial row
  __syncthreads();
  BcRows<D> cur;
  if (wid < n_it) bc_load_rows<D>(Qb, ent, wid, cnt, lg_tpw, slot, lane_off, hl, spare, cur);  // in flight while the block is staged
  for (int k0 = kbeg; k0 < kend; k0 += KSEG) {
    const int nk = min(KSEG, kend - k0), last = (nk - 1) >> 5;
    if (k0 > kbeg) {
      __syncthreads();  // every wavefront is done with the previous segment
      if (wid < n_it) bc_load_rows<D>(Qb, ent, wid, cnt, lg_tpw, slot, lane_off, hl, spare, cur);
    }
    t32_stage2<D, false, 64 * NW>(a.v.Ks + (size_t)g * D, a.v.Vs + (size_t)g * D, kstride, k0, nk, Kt, Vt);
    t32_write_tail(tail, nk - 32 * last);
    wait_loads();  // (so that the step loop is entered with no load outstanding and its waits count what an iteration leaves)
    __syncthreads();
    const bool fresh = k0 == kbeg;
    const lds_cptr klast = kl + last * T::BYTES, vlast = vl + last * T::BYTES;
    for (int it = wid; it < n_it; it += NW) {
      const uint32_t prow = cur.prow;
      T32State<D, SumParts> st;
      if (!fresh) bc_pick_up<D>(a, prow, spare, st);
#pragma unroll
      for (int t = 0; t < MAXT - 1; ++t)
        if (t < last) {
          const f32x16 s = t32_scores<D, false>(cur.qop, kl + t * T::BYTES, ln, splat16(0.f));
          if (t == 0 && fresh) t32_softmax<D, false, true>(st, s, vl, ln, sl2);
          else t32_softmax<D, false, false>(st, s, vl + t * T::BYTES, ln, sl2);
        }
      {
        const f32x16 s = t32_scores<D, false>(cur.qop, klast, ln, t32_tail(tail));
        // the query rows are done with: those of the next step take their registers
        if (it + NW < n_it) bc_load_rows<D>(Qb, ent, it + NW, cnt, lg_tpw, slot, lane_off, hl, spare, cur);
        if (last == 0 && fresh) t32_softmax<D, false, true>(st, s, vlast, ln, sl2);
        else t32_softmax<D, false, false>(st, s, vlast, ln, sl2);
      }
      // (a vote of the chunk's own columns: taken or not, the path decides how their probabilities are rounded)
      if (__builtin_expect(__any(prow != spare && !t32_in_range(st)), 0)) {
        BcRows<D> r;
        bc_load_rows<D>(Qb, ent, it, cnt, lg_tpw, slot, lane_off, hl, spare, r);
        if (fresh) t32_clear(st);
        else bc_pick_up<D>(a, prow, spare, st);
#pragma unroll 1
        for (int t = 0; t <= last; ++t) {
          const f32x16 s = t32_scores<D, false>(r.qop, kl + t * T::BYTES, ln, t < last ? splat16(0.f) : t32_tail(tail));
          t32_softmax_running<D, false>(st, s, vl + t * T::BYTES, ln, sl2);
        }
      }
      t32_store_rows<D>(a.po, prow, st.o);
      *reinterpret_cast<float2 *>(a.pml + (size_t)prow * 2) = make_float2(st.m, st.l.total());  // (both lanes of a column: the same)
    }
  }
}

// Merge of the per-block partials of the selection branch (the online-softmax recurrence of Algorithm 1 applied across
// blocks instead of key tiles), and the gate-weighted sum of eq. (4) in the same pass: one thread per (token, query
// head, 8 output dims).  Writes out_branch[1], lse[1] and out.
struct MergeArgs {
  const bf16_t *po;
  const float *pml;
  const int32_t *idx;
  const bf16_t *gates;
  bf16_t *Ob;  // [3,N,Hq,D]: branches 0 and 2 are read, 1 is written
  float *lse;  // [3,N,Hq]
  bf16_t *out;
  int N, Hq, Hkv, hs, T, D;
  SlcKeep keep;
};

// Blocks in a row of I: rows are ascending with the -1 padding at the end, and nearly all are full.
__device__ inline int selected(const int32_t *row, int T) {
  if (row[T - 1] >= 0) return T;
  int nv = 0;
  for (int j = 0; j < T; ++j) nv += row[j] >= 0 ? 1 : 0;
  return nv;
}

// FEW: up to 8 blocks a row, whose partials are requested before it is known how many there are (what lies in the other rows is not used).
template <bool FEW>
__global__ __launch_bounds__(256) void m_slc_merge(MergeArgs a) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int per_row = a.D / 8;
  if (i >= (size_t)a.N * a.Hq * per_row) return;
  const int c8 = (int)(i % per_row), h = (int)(i / per_row % a.Hq), tok = (int)(i / ((size_t)per_row * a.Hq));
  const int g = h / a.hs, hl = h % a.hs;
  const size_t slot0 = ((size_t)tok * a.Hkv + g) * a.T;
  float M = -INFINITY, L = 0.f, acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  auto add = [&](const float2 &ml, const bf16x8 &x) {
    const float wj = ml.x == -INFINITY ? 0.f : fast_exp2(ml.x - M);
    L += wj * ml.y;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += wj * (float)x[e];
  };
  if constexpr (FEW) {
    float2 ml[8];
    bf16x8 x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const size_t r = (slot0 + min(j, a.T - 1)) * a.hs + hl;
      ml[j] = *reinterpret_cast<const float2 *>(a.pml + r * 2);
      x[j] = ld8(a.po + r * a.D + 8 * c8);
    }
    const int nv = selected(a.idx + slot0, a.T);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (j < nv) M = fmaxf(M, ml[j].x);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (j < nv) add(ml[j], x[j]);
  } else {
    const int nv = selected(a.idx + slot0, a.T);
#pragma unroll 8
    for (int j = 0; j < nv; ++j) M = fmaxf(M, a.pml[((slot0 + j) * a.hs + hl) * 2]);
#pragma unroll 8
    for (int j = 0; j < nv; ++j) {
      const size_t r = (slot0 + j) * a.hs + hl;
      add(*reinterpret_cast<const float2 *>(a.pml + r * 2), ld8(a.po + r * a.D + 8 * c8));
    }
  }
  const float inv = L > 0.f ? 1.0f / L : 0.f;
  const size_t th = (size_t)tok * a.Hq + h, NH = (size_t)a.N * a.Hq;
  const size_t off = th * a.D + 8 * c8;
  bf16x8 os;
#pragma unroll
  for (int e = 0; e < 8; ++e) os[e] = (__bf16)(acc[e] * inv);
  if (a.keep.branch) *reinterpret_cast<bf16x8 *>(a.Ob + NH * a.D + off) = os;
  if (a.keep.lse && c8 == 0) a.lse[NH + th] = L > 0.f ? (M + __log2f(L)) * LN2 : -INFINITY;
  const float w0 = bf16_to_f32(a.gates[th * 3]), w1 = bf16_to_f32(a.gates[th * 3 + 1]), w2 = bf16_to_f32(a.gates[th * 3 + 2]);
  const bf16x8 x0 = ld8(a.Ob + off), x2 = ld8(a.Ob + 2 * NH * a.D + off);
  bf16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (__bf16)(w0 * (float)x0[e] + w1 * (float)os[e] + w2 * (float)x2[e]);
  *reinterpret_cast<bf16x8 *>(a.out + off) = o;
}

// ---------------------------------------------------------------------------------------------------------
// dQ of the selection branch where it does not go with dK and dV (slc_bwd_two_kernels), block-centric: the same exchange of
// loops as the forward kernel m_slc_fwd_bc, with the same tiles of 32 keys x 32 columns.  A workgroup
// holds one selection block's K and V rows in LDS and runs through a chunk of the tokens that selected it; every
// wavefront takes 32/h_s tokens per step on its own (query and dO rows in registers, no barrier, no column that did
// not select the block).  One bf16 partial dQ per (token, KV head, selected block) goes to memory; m_dq_merge adds them
// in rank order onto the fp32 compression + window part.  153k tokens, heads of 128: 13.9 -> 11.8 ms (16 columns before).
// ---------------------------------------------------------------------------------------------------------
struct BcDqArgs {
  MfmaView v;
  const bf16_t *Qs, *dOs;             // [N(pos)][Hq][D] sorted copies: Q, and the selection gate times dO
  const float *lse2s, *deltas;        // selection branch: [N(pos)][Hq]
  const int32_t *sel_list, *chunk_start;
  const uint8_t *sel_rank;
  const ChunkRef *chunk_order;
  bf16_t *pdq;                        // [N(pos)][Hkv][T][hs][D] and a spare row
};

template <int D>
struct BcDqRows {
  bf16x8 qop[D / 16], dop[D / 16];
  float lse2, nd;   // lse in log2 units; -delta (delta = gate * <dO, O>)
  uint32_t prow;    // ((pos*Hkv + g)*T + rank)*hs + head, or the spare row
};

template <int D>
__device__ inline void bc_dq_load_rows(const BcDqArgs &a, const int *tl, const int *sl, int step, int cnt, int g, BcDqRows<D> &r) {
  const int n = threadIdx.x & 31, h = threadIdx.x >> 5 & 1;
  const int hs = a.v.hs, hl = n % hs;
  const int e = step * (32 / hs) + n / hs;
  const int pos = tl[min(e, cnt - 1)], rank = sl[min(e, cnt - 1)];
  const uint32_t th = (uint32_t)pos * a.v.Hq + g * hs + hl;
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) {
    r.qop[ks] = ld8(a.Qs + (size_t)th * D + 8 * h + 16 * ks);
    r.dop[ks] = ld8(a.dOs + (size_t)th * D + 8 * h + 16 * ks);
  }
  r.lse2 = a.lse2s[th];
  r.nd = -a.deltas[th];
  r.prow = e < cnt ? (((uint32_t)pos * a.v.Hkv + g) * a.v.T + rank) * hs + hl : (uint32_t)((size_t)a.v.N * a.v.Hq * a.v.T);
}

// One 32-key LDS tile: transposed scores (K rows) and dP (V rows, against gate * dO; the accumulators start from
// -delta of their column, so the matrix instruction leaves dP - delta), dS^T = P (dP - delta), then dQ^T += K^T dS^T
// with K^T read from the same K tile through the transposing LDS load.  The softmax scale of dS is applied by the merge
// kernel, once per output element.
template <int D>
__device__ inline void bc_dq_scores(const BcDqRows<D> &r, lds_cptr kt, lds_cptr vt, const typename T32<D, false>::Lanes &ln, f32x16 &s,
                                    f32x16 &dp) {
  using T = T32<D, false>;
  dp = splat16(r.nd);
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) {
    s = mfma32(T::row(kt, ln, ks), r.qop[ks], s);
    dp = mfma32(T::row(vt, ln, ks), r.dop[ks], dp);
  }
}
template <int D, bool FIRST = false>
__device__ inline void bc_dq_tile(f32x16 (&acc)[D / 32], const f32x16 &s, const f32x16 &dp, lds_cptr kt,
                                  const typename T32<D, false>::Lanes &ln, float lse2, float sl2) {
#pragma unroll
  for (int kc = 0; kc < 2; ++kc) {
    bf16x8 ds;
#pragma unroll
    for (int j = 0; j < 8; ++j)  // dp = gate * dP - delta: the dO rows are gate * dO
      ds[j] = (__bf16)(fast_exp2(__builtin_fmaf(s[8 * kc + j], sl2, -lse2)) * dp[8 * kc + j]);
#pragma unroll
    for (int db = 0; db < D / 32; ++db) acc[db] = mfma32(T32<D, false>::tr(kt, ln, db, kc), ds, FIRST && kc == 0 ? splat16(0.f) : acc[db]);
  }
}

template <int D, int NW, int KSEG, int WPE>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(WPE))) void m_bwd_dq_bc(BcDqArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  using T = T32<D, false>;
  constexpr int MAXT = KSEG / 32;
  unsigned char *Kt = smem, *Vt = Kt + MAXT * T::BYTES;
  int *tl = (int *)(Vt + MAXT * T::BYTES), *sl = tl + BC_CHUNK;
  float *tail = (float *)(sl + BC_CHUNK);
  const int wid = uniform(threadIdx.x >> 6);
  const int hs = a.v.hs, Hkv = a.v.Hkv, Ns = a.v.Ns;
  const int wi = blockIdx.x;
  if (wi >= a.chunk_start[Hkv * Ns]) return;
  const ChunkRef cr = a.chunk_order[wi];
  const int key = uniform(cr.key), g = key / Ns, blk = key % Ns;
  const int kbeg = uniform(a.v.slc_start[blk]), kend = uniform(a.v.slc_start[blk + 1]);
  const int qbeg = uniform(cr.first), cnt = uniform(cr.count);
  // the chunk's tokens (sorted positions) and the rank of this block in each token's row of I
  for (int i = threadIdx.x; i < cnt; i += 64 * NW) {
    tl[i] = a.sel_list[qbeg + i];
    sl[i] = a.sel_rank[qbeg + i];
  }
  const int tpw = 32 / hs;
  const int n_it = (cnt + tpw - 1) / tpw;
  const uint32_t kstride = (uint32_t)(Hkv * D), spare = (uint32_t)((size_t)a.v.N * a.v.Hq * a.v.T);  // behind the last partial row
  const float sl2 = in_vgpr(a.v.sl2);
  const typename T::Lanes ln = T::lanes();
  const lds_cptr kt = (lds_cptr)Kt, vt = (lds_cptr)Vt;
  __syncthreads();
  BcDqRows<D> cur;
  if (wid < n_it) bc_dq_load_rows<D>(a, tl, sl, wid, cnt, g, cur);
  for (int k0 = kbeg; k0 < kend; k0 += KSEG) {
    const int nk = min(KSEG, kend - k0), last = (nk - 1) >> 5;
    if (k0 > kbeg) {
      __syncthreads();
      if (wid < n_it) bc_dq_load_rows<D>(a, tl, sl, wid, cnt, g, cur);
    }
    t32_stage2<D, false, 64 * NW>(a.v.Ks + (size_t)g * D, a.v.Vs + (size_t)g * D, kstride, k0, nk, Kt, Vt);
    t32_write_tail(tail, nk - 32 * last);
    wait_loads();  // (so that the step loop is entered with no load outstanding and its waits count what an iteration leaves)
    __syncthreads();
    const lds_cptr klast = kt + last * T::BYTES, vlast = vt + last * T::BYTES;
    for (int it = wid; it < n_it; it += NW) {
      const uint32_t prow = cur.prow;
      const float lse2 = cur.lse2;
      f32x16 acc[D / 32];
      const bool fresh = k0 == kbeg;
      if (!fresh) {  // continue from the partial of the earlier segments (columns past the end of the chunk: from nothing)
        if (prow != spare) bc_pick_up_row<D>(a.pdq, prow, acc);
        else
#pragma unroll
          for (int db = 0; db < D / 32; ++db) acc[db] = splat16(0.f);
      }
#pragma unroll
      for (int t = 0; t < MAXT - 1; ++t)
        if (t < last) {
          f32x16 s = splat16(0.f), dp;
          bc_dq_scores<D>(cur, kt + t * T::BYTES, vt + t * T::BYTES, ln, s, dp);
          if (t == 0 && fresh) bc_dq_tile<D, true>(acc, s, dp, kt, ln, lse2, sl2);
          else bc_dq_tile<D>(acc, s, dp, kt + t * T::BYTES, ln, lse2, sl2);
        }
      {
        f32x16 s = t32_tail(tail), dp;
        bc_dq_scores<D>(cur, klast, vlast, ln, s, dp);
        // the rows are done with: those of the next step take their registers
        if (it + NW < n_it) bc_dq_load_rows<D>(a, tl, sl, it + NW, cnt, g, cur);
        if (last == 0 && fresh) bc_dq_tile<D, true>(acc, s, dp, klast, ln, lse2, sl2);
        else bc_dq_tile<D>(acc, s, dp, klast, ln, lse2, sl2);
      }
      t32_store_rows<D>(a.pdq, prow, acc);
    }
  }
}

// dQ[tok] = (compression + window part, fp32, by sorted position) + scale * sum over the token's selected blocks, in
// rank order, of the partial dQ (which the block-centric kernel leaves without the softmax scale).  One thread per
// (sorted position, query head, 8 dims).
struct DqMergeArgs {
  const bf16_t *pdq;
  const float *dQp;
  const int32_t *idx, *perm;
  bf16_t *dQ;
  int N, Hq, Hkv, hs, T, D;
  float scale;
};

__global__ __launch_bounds__(256) void m_dq_merge(DqMergeArgs a) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int per_row = a.D / 8;
  if (i >= (size_t)a.N * a.Hq * per_row) return;
  const int c8 = (int)(i % per_row), h = (int)(i / per_row % a.Hq), pos = (int)(i / ((size_t)per_row * a.Hq));
  const int g = h / a.hs, hl = h % a.hs, tok = a.perm[pos];
  const int nv = selected(a.idx + ((size_t)tok * a.Hkv + g) * a.T, a.T);
  const float *base = a.dQp + ((size_t)pos * a.Hq + h) * a.D + 8 * c8;
  const float4 b0 = *reinterpret_cast<const float4 *>(base), b1 = *reinterpret_cast<const float4 *>(base + 4);
  const float part[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const size_t slot0 = ((size_t)pos * a.Hkv + g) * a.T;
#pragma unroll 4
  for (int j = 0; j < nv; ++j) {
    const bf16x8 x = ld8(a.pdq + ((slot0 + j) * a.hs + hl) * a.D + 8 * c8);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += (float)x[e];
  }
  bf16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (__bf16)__builtin_fmaf(a.scale, acc[e], part[e]);
  *reinterpret_cast<bf16x8 *>(a.dQ + ((size_t)tok * a.Hq + h) * a.D + 8 * c8) = o;
}

// dQ: wavefronts per workgroup, keys held in LDS at a time.
constexpr int DQ_WAVES = 8, DQ_KSEG = 256;
template <int D> constexpr int dq_wpe() { return D == 32 ? 4 : 2; }
// Forward: wavefronts per workgroup and per SIMD, keys in LDS at a time (see m_slc_fwd_bc for the figures).
template <int D> struct BcFwdShape { static constexpr int NW = 8, KSEG = 256, WPE = 4; };
template <> struct BcFwdShape<128> { static constexpr int NW = 8, KSEG = 256, WPE = 2; };

// upper bound of the number of chunks: every (KV head, block) list adds at most one partly filled chunk
unsigned chunk_bound(const MfmaView &v, int chunk_len) {
  const size_t entries = (size_t)v.N * v.Hkv * v.T;
  return (unsigned)(entries / chunk_len + (size_t)v.Hkv * v.Ns);
}

template <int D>
int launch_slc_forward(const MfmaView &v, const bf16_t *q, const SelIndex &sel, const SlcPartials &part,
                       hipStream_t s) {
  using BS = BcFwdShape<D>;
  auto kernel = m_slc_fwd_bc<D, BS::NW, BS::KSEG, BS::WPE>;
  static std::once_flag once;  // raise the dynamic LDS limit once per process for this instantiation
  std::call_once(once, [&] {
    (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  });
  BcFwdArgs b{v, q, sel.list, sel.bc_chunk_start, sel.rank, sel.bc_order, part.o, part.ml};
  kernel<<<dim3(chunk_bound(v, sel.bc_chunk_len)), 64 * BS::NW, bc_lds_bytes<D, BS::KSEG>(), s>>>(b);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}

template <int D>
int launch_slc_dq(const MfmaView &v, const BwdBuffers &w, hipStream_t s) {
  static std::once_flag once;
  std::call_once(once, [] {
    (void)hipFuncSetAttribute((const void *)m_bwd_dq_bc<D, DQ_WAVES, DQ_KSEG, dq_wpe<D>()>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              160 * 1024);
  });
  const size_t NH = (size_t)v.N * v.Hq;
  BcDqArgs b{v, w.Qs, w.dOg + NH * D, w.lse2s + NH, w.deltag + NH, w.sel.list, w.sel.bc_chunk_start, w.sel.rank, w.sel.bc_order, w.part.o};
  m_bwd_dq_bc<D, DQ_WAVES, DQ_KSEG, dq_wpe<D>()><<<dim3(chunk_bound(v, w.sel.bc_chunk_len)), 64 * DQ_WAVES, bc_lds_bytes<D, DQ_KSEG>(), s>>>(b);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}

}  // namespace

int slc_forward_kernel(const MfmaView &v, int D, const void *q, const SelIndex &sel,
                       const SlcPartials &part, hipStream_t s) {
  switch (D) {
    case 32: return launch_slc_forward<32>(v, (const bf16_t *)q, sel, part, s);
    case 64: return launch_slc_forward<64>(v, (const bf16_t *)q, sel, part, s);
    case 128: return launch_slc_forward<128>(v, (const bf16_t *)q, sel, part, s);
    default: return SSA_ERR_UNSUPPORTED;
  }
}

int slc_merge_kernel(const MfmaView &v, int D, const SlcPartials &part, const int32_t *idx, const void *gates,
                     void *out_branch, float *lse, void *out, SlcKeep keep, hipStream_t s) {
  MergeArgs m{part.o, part.ml, idx, (const bf16_t *)gates, (bf16_t *)out_branch, lse, (bf16_t *)out,
              v.N, v.Hq, v.Hkv, v.hs, v.T, D, keep};
  const size_t threads = (size_t)v.N * v.Hq * (D / 8);
  // Small problems wait for one round trip to memory instead of two.  Whole forward, one after the other / together, us: 1k tokens, top-8 59.0 / 57.0,
  // 5k, top-4 100.3 / 98.1, 11k, top-8 267.8 / 264.8, 8k, heads of 128 338.6 / 333.8; with two blocks a row the eight requests are too many (11k
  // 172.5 / 177.3), and in large ones the registers cost wavefronts (40k 1210 / 1215).
  const bool few = v.T >= 4 && v.T <= 8 && (size_t)v.N * v.Hq * v.T <= (size_t)1 << 21;
  (few ? m_slc_merge<true> : m_slc_merge<false>)<<<(unsigned)((threads + 255) / 256), 256, 0, s>>>(m);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}

int slc_dq_kernel(const MfmaView &v, int D, const BwdBuffers &w, hipStream_t s) {
  switch (D) {
    case 32: return launch_slc_dq<32>(v, w, s);
    case 64: return launch_slc_dq<64>(v, w, s);
    case 128: return launch_slc_dq<128>(v, w, s);
    default: return SSA_ERR_UNSUPPORTED;
  }
}

int slc_dq_merge_kernel(const MfmaView &v, int D, const BwdBuffers &w, const int32_t *idx, void *dq, hipStream_t s) {
  DqMergeArgs m{w.part.o, w.dQp, idx, v.perm, (bf16_t *)dq, v.N, v.Hq, v.Hkv, v.hs, v.T, D, v.scale};
  const size_t threads = (size_t)v.N * v.Hq * (D / 8);
  m_dq_merge<<<(unsigned)((threads + 255) / 256), 256, 0, s>>>(m);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}
