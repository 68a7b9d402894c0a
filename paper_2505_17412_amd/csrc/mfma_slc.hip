// Selection branch of SSA on bf16 MFMA for gfx950, block-centric: Algorithm 1 with its two loops exchanged, forward and
// dQ, and the kernels that merge the per-block partial results (the forward one also forms the gated sum of eq. (4)).
// A translation unit of its own: these kernels have no barrier in their inner loops and long straight-line tile code,
// and are compiled with an instruction scheduler setting of their own (see build.py).
#include "mfma_common.h"
#include "mfma_launch.h"
#include "mfma_qc.h"
#include "mfma_bc.h"

#include <mutex>

namespace {

// ---------------------------------------------------------------------------------------------------------
// Selection branch, block-centric (Algorithm 1 with the loops exchanged): the outer loop runs over the selected blocks,
// the inner one over the query tokens that selected the block.  A workgroup takes one (KV head, selection block) and a
// chunk of up to BC_CHUNK tokens of that block's selector list, puts the block's K and V rows into LDS ONCE (up to KSEG
// keys; longer blocks in several segments) and lets every wavefront run, on its own and without any barrier, through
// groups of CB*16/h_s tokens: all CB*16 query columns of a matrix tile then take part in every key tile (nothing is
// computed for a token that did not select the block), the K and V^T operands read from LDS feed CB column blocks,
// and no wavefront waits for another.  The price is one partial result per (token, KV head, selected block): the
// unnormalised output in bf16 with its running maximum and sum (Algorithm 1's o, m, l for that block alone), merged per
// token afterwards (m_slc_merge).  A wavefront that meets a block longer than KSEG picks its own partial up again for
// the next segment.
// Bound: the sum of matrix and vector issue (a synthetic copy of one 16-column tile with its LDS reads takes 116 ns per SIMD
// at four wavefronts, of which this kernel's tiles and steps take 145), and for short blocks the partial rows going out.
// One column block at head_dim 64 (128 registers, four wavefronts per SIMD; two blocks at two or four wavefronts: 1111 and
// 1038 us against 989), two at head_dim 128, where the accumulators leave two wavefronts anyway.  62k tokens, 16 heads of
// 64, top-16: 1090 -> 990 us (no maximum and no rescaling after the first tile, chunk entries prepared in LDS, list entries
// and chunk bounds read directly); 153k tokens, heads of 128: 12.4 -> 11.3 ms; blocks of 64 keys (sequences): 807 -> 738 us
// with whole-line stores.
// ---------------------------------------------------------------------------------------------------------
struct BcFwdArgs {
  MfmaView v;
  const bf16_t *Q;
  const int32_t *sel_list, *chunk_start;  // lists of caller indices
  const uint8_t *sel_rank;
  const ChunkRef *chunk_order;
  bf16_t *po;  // [N][Hkv][T][hs][D]
  float *pml;  // [N][Hkv][T][hs][2]
};

// LDS plan (bytes): K tiles | V tiles (KSEG/32 tiles each, PTile layout) | chunk entries [BC_CHUNK][2]
template <int D, int KSEG>
constexpr size_t bc_lds_bytes() { return (size_t)2 * (KSEG / 32) * PTile<D, false>::BYTES + (size_t)2 * BC_CHUNK * sizeof(int); }

// Query operands and partial-row index of one wavefront step: column n of column block cb stands for chunk entry
// (step*CB + cb)*(16/h_s) + n/h_s, head n % h_s of the KV group.  Columns past the end of the chunk repeat its last entry
// and are not stored.
template <int D, int CB>
struct BcRows {
  bf16x8 qop[CB][D / 32];
  uint32_t prow[CB];  // ((tok*Hkv + g)*T + rank)*hs + head: row of the partial arrays (below 2^32: N*Hq*T is)
  bool valid[CB];
};

// qoff, prow0: per chunk entry the byte offset of the token's query rows of this KV group and its first partial row.
template <int D, int CB>
__device__ inline void bc_load_rows(const unsigned char *Q, const uint2 *ent, int step, int cnt, int lg_tpw, int slot, uint32_t lane_off,
                                    int hl, BcRows<D, CB> &r) {
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    const int e = ((step * CB + cb) << lg_tpw) + slot;
    r.valid[cb] = e < cnt;
    const uint2 x = ent[min(e, cnt - 1)];
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks) r.qop[cb][ks] = *reinterpret_cast<const bf16x8 *>(Q + (x.x + lane_off) + 64 * ks);
    r.prow[cb] = x.y + hl;
  }
}

// Scores of CB blocks of 16 query columns over one 32-key LDS tile: v[j] = key 8*quad + j of the tile, column n.
template <int D, int CB>
__device__ inline void bc_scores(const bf16x8 (&qop)[CB][D / 32], lds_cptr kt, const typename PTile<D, false>::Lanes &ln, float (&v)[CB][8]) {
  f32x4 s[CB][2];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) s[cb][0] = s[cb][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < D / 32; ++ks)
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      const bf16x8 k = p_row_operand<D, false>(kt, ln, sub, ks);
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) s[cb][sub] = mfma16(k, qop[cb][ks], s[cb][sub]);
    }
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int j = 0; j < 8; ++j) v[cb][j] = s[cb][j >> 2][j & 3];
}

// One step of the softmax (Algorithm 1, inner loop body) over one tile.  The reference exponent of a column is the maximum
// of its first tile (FIRST; log2 units, st.m) and stays: later tiles cost a fused multiply-add, an exponential and half a
// conversion per score, no maximum and no rescaling.  The result does not depend on the reference as long as nothing leaves
// the range of the floats, which the caller checks on the finished sums (bc_in_range).
// MASK: only the first `left` keys of the tile exist.
template <int D, int CB, bool MASK, bool FIRST>
__device__ inline void bc_fwd_tile(FwdState<D, CB> &st, const bf16x8 (&qop)[CB][D / 32], lds_cptr kt, lds_cptr vt,
                                   const typename PTile<D, false>::Lanes &ln, int left, float sl2, const bf16x8 &ones) {
  float v[CB][8];
  bc_scores<D, CB>(qop, kt, ln, v);
  if (MASK) {
    const int first = 8 * (int)(threadIdx.x >> 4 & 3);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (first + j >= left) v[cb][j] = -INFINITY;
  }
  if (FIRST) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const float(&x)[8] = v[cb];
      st.m[cb] = column_max(fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])))) * sl2;
    }
  }
  bf16x8 pb[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
    for (int j = 0; j < 8; ++j) pb[cb][j] = (__bf16)fast_exp2(__builtin_fmaf(v[cb][j], sl2, -st.m[cb]));
    // the normaliser on the matrix pipe: an all-ones A operand sums the 32 probabilities of every column, in the same bf16
    // rounding the numerator uses, and leaves the total in every lane of the column
    st.l[cb] = mfma16(ones, pb[cb], st.l[cb]);
  }
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) {
    const bf16x8 av = p_tr_operand<D, false>(vt, ln, dt);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) st.o[cb][dt] = mfma16(av, pb[cb], st.o[cb][dt]);
  }
}

// The first tile's maximum contributes 1 to the sum, so nothing that counts is lost below; a sum under 2^60 leaves room for
// values of the same size.
__device__ inline bool bc_in_range(float l) { return l < 0x1p60f; }

// The same step with a running maximum (raised lazily, see fwd_tile): what a column whose scores rise far above its first
// tile's goes through instead.  st.m in log2 units.
template <int D>
__device__ inline void bc_fwd_tile_safe(FwdState<D, 1> &st, const bf16x8 (&qop)[1][D / 32], lds_cptr kt, lds_cptr vt,
                                        const typename PTile<D, false>::Lanes &ln, int left, float sl2, const bf16x8 &ones) {
  float v[1][8];
  bc_scores<D, 1>(qop, kt, ln, v);
  const int first = 8 * (int)(threadIdx.x >> 4 & 3);
  float pm = -INFINITY;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    v[0][j] = first + j < left ? v[0][j] * sl2 : -INFINITY;
    pm = fmaxf(pm, v[0][j]);
  }
  if (__any(pm > st.m[0] + 8.f)) {
    float tmax = fmaxf(pm, __shfl_xor(pm, 16));
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
    const float mn = fmaxf(st.m[0], tmax);
    const float alpha = mn == -INFINITY ? 1.0f : fast_exp2(st.m[0] - mn);
    st.l[0][0] *= alpha;
    st.m[0] = mn;
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) st.o[0][dt] *= alpha;
  }
  const float neg = st.m[0] != -INFINITY ? -st.m[0] : -INFINITY;
  bf16x8 pb;
#pragma unroll
  for (int j = 0; j < 8; ++j) pb[j] = (__bf16)fast_exp2(v[0][j] + neg);
  st.l[0] = mfma16(ones, pb, st.l[0]);
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) st.o[0][dt] = mfma16(p_tr_operand<D, false>(vt, ln, dt), pb, st.o[0][dt]);
}

// Partial of the earlier segments of a long block, picked up again.
template <int D>
__device__ inline void bc_pick_up(const BcFwdArgs &a, uint32_t prow, bool valid, f32x4 (&o)[D / 16], f32x4 &l, float &m) {
  const int quad = threadIdx.x >> 4 & 3;
  m = 0.f;
  if (!valid) return;
  const float2 ml = *reinterpret_cast<const float2 *>(a.pml + (size_t)prow * 2);
  m = ml.x;
  l[0] = ml.y;
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) {
    const bf16x4 x = *reinterpret_cast<const bf16x4 *>(a.po + (size_t)prow * D + acc_dim(dt, quad));
#pragma unroll
    for (int i = 0; i < 4; ++i) o[dt][i] = (float)x[i];
  }
}

template <int D, int CB, int NW, int KSEG, int WPE>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(WPE))) void m_slc_fwd_bc(BcFwdArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  using P = PTile<D, false>;
  constexpr int MAXT = KSEG / 32;
  unsigned char *Kt = smem, *Vt = Kt + MAXT * P::BYTES;
  uint2 *ent = (uint2 *)(Vt + MAXT * P::BYTES);
  const int wid = threadIdx.x >> 6, quad = threadIdx.x >> 4 & 3, n = threadIdx.x & 15;
  const int hs = a.v.hs, Hkv = a.v.Hkv, Ns = a.v.Ns;
  const int wi = bc_chunk_of_workgroup(a.chunk_start[Hkv * Ns]);
  if (wi < 0) return;
  const ChunkRef cr = a.chunk_order[wi];
  const int g = cr.key / Ns, blk = cr.key % Ns;
  const int kbeg = a.v.slc_start[blk], kend = a.v.slc_start[blk + 1];
  const int qbeg = cr.first, cnt = cr.count;
  for (int i = threadIdx.x; i < cnt; i += 64 * NW) {
    const uint32_t tok = (uint32_t)a.sel_list[qbeg + i];
    ent[i] = make_uint2((tok * a.v.Hq + g * hs) * (D * 2), ((tok * Hkv + g) * a.v.T + a.sel_rank[qbeg + i]) * hs);
  }
  const int lg_tpw = 31 - __builtin_clz(16 / hs), slot = n / hs, hl = n % hs;
  const uint32_t lane_off = (uint32_t)(hl * D * 2 + 16 * quad);
  const unsigned char *Qb = (const unsigned char *)a.Q;
  const int n_it = (cnt + (CB << lg_tpw) - 1) / (CB << lg_tpw);
  const uint32_t kstride = (uint32_t)(Hkv * D);
  const float sl2 = a.v.sl2;
  const bf16x8 ones = ones_operand();
  const typename P::Lanes ln = P::lanes();
  const lds_cptr kl = (lds_cptr)Kt, vl = (lds_cptr)Vt;
  __syncthreads();
  BcRows<D, CB> cur;
  if (wid < n_it) bc_load_rows<D, CB>(Qb, ent, wid, cnt, lg_tpw, slot, lane_off, hl, cur);  // in flight while the block is staged
  for (int k0 = kbeg; k0 < kend; k0 += KSEG) {
    const int nk = min(KSEG, kend - k0), nfull = nk >> 5;
    if (k0 > kbeg) {
      __syncthreads();  // every wavefront is done with the previous segment
      if (wid < n_it) bc_load_rows<D, CB>(Qb, ent, wid, cnt, lg_tpw, slot, lane_off, hl, cur);
    }
    p_stage2<D, false, 64 * NW>(a.v.Ks + (size_t)g * D, a.v.Vs + (size_t)g * D, kstride, k0, (nk + 31) >> 5, Kt, Vt);
    __syncthreads();
    for (int it = wid; it < n_it; it += NW) {
      BcRows<D, CB> nxt;  // the next step's operands are requested before this step's arithmetic
      if (it + NW < n_it) bc_load_rows<D, CB>(Qb, ent, it + NW, cnt, lg_tpw, slot, lane_off, hl, nxt);
      FwdState<D, CB> st;
      init_state(st);
      const bool fresh = k0 == kbeg;
      if (!fresh)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) bc_pick_up<D>(a, cur.prow[cb], cur.valid[cb], st.o[cb], st.l[cb], st.m[cb]);
      if (fresh && nfull > 0) bc_fwd_tile<D, CB, false, true>(st, cur.qop, kl, vl, ln, 32, sl2, ones);
      else if (fresh) bc_fwd_tile<D, CB, true, true>(st, cur.qop, kl, vl, ln, nk, sl2, ones);
      else if (nfull > 0) bc_fwd_tile<D, CB, false, false>(st, cur.qop, kl, vl, ln, 32, sl2, ones);
#pragma unroll
      for (int t = 1; t < MAXT; ++t)
        if (t < nfull) bc_fwd_tile<D, CB, false, false>(st, cur.qop, kl + t * P::BYTES, vl + t * P::BYTES, ln, 32, sl2, ones);
      if ((nk & 31) && (nfull > 0 || !fresh))
        bc_fwd_tile<D, CB, true, false>(st, cur.qop, kl + nfull * P::BYTES, vl + nfull * P::BYTES, ln, nk & 31, sl2, ones);
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        if (__builtin_expect(__any(cur.valid[cb] && !bc_in_range(st.l[cb][0])), 0)) {
          FwdState<D, 1> safe;
          init_state(safe);
          bf16x8 q1[1][D / 32];
#pragma unroll
          for (int ks = 0; ks < D / 32; ++ks) q1[0][ks] = cur.qop[cb][ks];
          if (k0 > kbeg) bc_pick_up<D>(a, cur.prow[cb], cur.valid[cb], safe.o[0], safe.l[0], safe.m[0]);
#pragma unroll 1
          for (int t = 0; t < (nk + 31) >> 5; ++t)
            bc_fwd_tile_safe<D>(safe, q1, kl + t * P::BYTES, vl + t * P::BYTES, ln, nk - 32 * t, sl2, ones);
          st.m[cb] = safe.m[0];
          st.l[cb] = safe.l[0];
#pragma unroll
          for (int dt = 0; dt < D / 16; ++dt) st.o[cb][dt] = safe.o[0][dt];
        }
        // (a column past the end of the chunk repeats the chunk's last entry and is not stored)
        store_partial_row<D>(a.po, cur.prow[cb], st.o[cb], cur.valid[cb]);
        if (cur.valid[cb] && quad == 0)
          *reinterpret_cast<float2 *>(a.pml + (size_t)cur.prow[cb] * 2) = make_float2(st.m[cb], st.l[cb][0]);
      }
      cur = nxt;
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
};

__global__ __launch_bounds__(256) void m_slc_merge(MergeArgs a) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int per_row = a.D / 8;
  if (i >= (size_t)a.N * a.Hq * per_row) return;
  const int c8 = (int)(i % per_row), h = (int)(i / per_row % a.Hq), tok = (int)(i / ((size_t)per_row * a.Hq));
  const int g = h / a.hs, hl = h % a.hs;
  const size_t slot0 = ((size_t)tok * a.Hkv + g) * a.T;
  const int32_t *row = a.idx + slot0;
  int nv = 0;  // rows are ascending with the -1 padding at the end
  for (int j = 0; j < a.T; ++j) nv += row[j] >= 0 ? 1 : 0;
  float M = -INFINITY;
  for (int j = 0; j < nv; ++j) M = fmaxf(M, a.pml[((slot0 + j) * a.hs + hl) * 2]);
  float L = 0.f, acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int j = 0; j < nv; ++j) {
    const size_t r = (slot0 + j) * a.hs + hl;
    const float2 ml = *reinterpret_cast<const float2 *>(a.pml + r * 2);
    const bf16x8 x = ld8(a.po + r * a.D + 8 * c8);
    const float wj = ml.x == -INFINITY ? 0.f : fast_exp2(ml.x - M);
    L += wj * ml.y;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += wj * (float)x[e];
  }
  const float inv = L > 0.f ? 1.0f / L : 0.f;
  const size_t th = (size_t)tok * a.Hq + h, NH = (size_t)a.N * a.Hq;
  const size_t off = th * a.D + 8 * c8;
  bf16x8 os;
#pragma unroll
  for (int e = 0; e < 8; ++e) os[e] = (__bf16)(acc[e] * inv);
  *reinterpret_cast<bf16x8 *>(a.Ob + NH * a.D + off) = os;
  if (c8 == 0) a.lse[NH + th] = L > 0.f ? (M + __log2f(L)) * LN2 : -INFINITY;
  const float w0 = bf16_to_f32(a.gates[th * 3]), w1 = bf16_to_f32(a.gates[th * 3 + 1]), w2 = bf16_to_f32(a.gates[th * 3 + 2]);
  const bf16x8 x0 = ld8(a.Ob + off), x2 = ld8(a.Ob + 2 * NH * a.D + off);
  bf16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (__bf16)(w0 * (float)x0[e] + w1 * (float)os[e] + w2 * (float)x2[e]);
  *reinterpret_cast<bf16x8 *>(a.out + off) = o;
}

// ---------------------------------------------------------------------------------------------------------
// dQ of the selection branch where it does not go with dK and dV (slc_bwd_two_kernels), block-centric: the same exchange of
// loops as the forward kernel m_slc_fwd_bc.  A workgroup
// holds one selection block's K and V rows in LDS and runs through a chunk of the tokens that selected it; every
// wavefront takes 16/h_s tokens per step on its own (query and dO rows in registers, no barrier, no column that did
// not select the block).  One bf16 partial dQ per (token, KV head, selected block) goes to memory; m_dq_merge adds them
// in rank order onto the fp32 compression + window part.
// ---------------------------------------------------------------------------------------------------------
struct BcDqArgs {
  MfmaView v;
  const bf16_t *Qs, *dOs;             // [N(pos)][Hq][D] sorted copies: Q, and the selection gate times dO
  const float *lse2s, *deltas;        // selection branch: [N(pos)][Hq]
  const int32_t *sel_list, *chunk_start;
  const uint8_t *sel_rank;
  const ChunkRef *chunk_order;
  bf16_t *pdq;                        // [N(pos)][Hkv][T][hs][D]
};

template <int D>
struct BcDqRows {
  bf16x8 qop[D / 32], dop[D / 32];
  float lse2, nd;   // lse in log2 units; -delta (delta = gate * <dO, O>)
  uint32_t prow;         // ((pos*Hkv + g)*T + rank)*hs + head
  bool valid;
};

template <int D>
__device__ inline void bc_dq_load_rows(const BcDqArgs &a, const int *tl, const int *sl, int step, int cnt, int g, BcDqRows<D> &r) {
  const int n = threadIdx.x & 15, quad = threadIdx.x >> 4 & 3;
  const int hs = a.v.hs, hl = n % hs;
  const int e = step * (16 / hs) + n / hs;
  r.valid = e < cnt;
  const int pos = r.valid ? tl[e] : 0, rank = r.valid ? sl[e] : 0;
  const size_t th = (size_t)pos * a.v.Hq + g * hs + hl;
#pragma unroll
  for (int ks = 0; ks < D / 32; ++ks) {
    r.qop[ks] = r.valid ? ld8(a.Qs + th * D + 8 * quad + 32 * ks) : zero8();
    r.dop[ks] = r.valid ? ld8(a.dOs + th * D + 8 * quad + 32 * ks) : zero8();
  }
  r.lse2 = r.valid ? a.lse2s[th] : INFINITY;  // a missing column gets P = exp2(-inf) = 0
  r.nd = -a.deltas[th];
  r.prow = (uint32_t)((((size_t)pos * a.v.Hkv + g) * a.v.T + rank) * hs + hl);
}

// One 32-key LDS tile: transposed scores (K rows) and dP (V rows, against gate * dO; the accumulators start from
// -delta of their column, so the matrix instruction leaves dP - delta), dS^T = P (dP - delta), then dQ^T += K^T dS^T
// with K^T read from the same K tile through the transposing LDS load.  The softmax scale of dS is applied by the merge
// kernel, once per output element.
template <int D, bool MASK>
__device__ inline void bc_dq_tile(f32x4 (&acc)[D / 16], const BcDqRows<D> &r, lds_cptr kt, lds_cptr vt,
                                  const typename PTile<D, false>::Lanes &ln, int key0, int nk, float sl2) {
  f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0, p0 = {r.nd, r.nd, r.nd, r.nd}, p1 = p0;
#pragma unroll
  for (int ks = 0; ks < D / 32; ++ks) {
    s0 = mfma16(p_row_operand<D, false>(kt, ln, 0, ks), r.qop[ks], s0);
    s1 = mfma16(p_row_operand<D, false>(kt, ln, 1, ks), r.qop[ks], s1);
    p0 = mfma16(p_row_operand<D, false>(vt, ln, 0, ks), r.dop[ks], p0);
    p1 = mfma16(p_row_operand<D, false>(vt, ln, 1, ks), r.dop[ks], p1);
  }
  bf16x8 ds;
  const int first = key0 + 8 * (int)(threadIdx.x >> 4 & 3);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float sv = j < 4 ? s0[j & 3] : s1[j & 3], dp = j < 4 ? p0[j & 3] : p1[j & 3];
    float p = fast_exp2(__builtin_fmaf(sv, sl2, -r.lse2));
    if (MASK && first + j >= nk) p = 0.f;
    ds[j] = (__bf16)(p * dp);  // dp = gate * dP - delta: the dO rows are gate * dO
  }
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) acc[dt] = mfma16(p_tr_operand<D, false>(kt, ln, dt), ds, acc[dt]);
}

template <int D, int KSEG>
constexpr size_t bc_dq_lds_bytes() { return (size_t)2 * (KSEG / 32) * PTile<D, false>::BYTES + (size_t)2 * BC_CHUNK * sizeof(int); }

template <int D, int NW, int KSEG>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D <= 64 ? 4 : 2))) void m_bwd_dq_bc(BcDqArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  using P = PTile<D, false>;
  constexpr int MAXT = KSEG / 32;
  unsigned char *Kt = smem, *Vt = Kt + MAXT * P::BYTES;
  int *tl = (int *)(Vt + MAXT * P::BYTES), *sl = tl + BC_CHUNK;
  const int wid = threadIdx.x >> 6, quad = threadIdx.x >> 4 & 3;
  const int hs = a.v.hs, Hkv = a.v.Hkv, Ns = a.v.Ns;
  const int wi = bc_chunk_of_workgroup(a.chunk_start[Hkv * Ns]);
  if (wi < 0) return;
  const ChunkRef cr = a.chunk_order[wi];
  const int g = cr.key / Ns, blk = cr.key % Ns;
  const int kbeg = a.v.slc_start[blk], kend = a.v.slc_start[blk + 1];
  const int qbeg = cr.first, cnt = cr.count;
  // the chunk's tokens (sorted positions) and the rank of this block in each token's row of I
  for (int i = threadIdx.x; i < cnt; i += 64 * NW) {
    tl[i] = a.sel_list[qbeg + i];
    sl[i] = a.sel_rank[qbeg + i];
  }
  const int tpw = 16 / hs;
  const int n_it = (cnt + tpw - 1) / tpw;
  const uint32_t kstride = (uint32_t)(Hkv * D);
  const float sl2 = a.v.sl2;
  const typename P::Lanes ln = P::lanes();
  const lds_cptr kt = (lds_cptr)Kt, vt = (lds_cptr)Vt;
  __syncthreads();
  BcDqRows<D> cur;
  if (wid < n_it) bc_dq_load_rows<D>(a, tl, sl, wid, cnt, g, cur);
  for (int k0 = kbeg; k0 < kend; k0 += KSEG) {
    const int nk = min(KSEG, kend - k0), nfull = nk >> 5;
    if (k0 > kbeg) {
      __syncthreads();
      if (wid < n_it) bc_dq_load_rows<D>(a, tl, sl, wid, cnt, g, cur);
    }
    p_stage2<D, false, 64 * NW>(a.v.Ks + (size_t)g * D, a.v.Vs + (size_t)g * D, kstride, k0, (nk + 31) >> 5, Kt, Vt);
    __syncthreads();
    for (int it = wid; it < n_it; it += NW) {
      BcDqRows<D> nxt;
      if (it + NW < n_it) bc_dq_load_rows<D>(a, tl, sl, it + NW, cnt, g, nxt);
      f32x4 acc[D / 16];
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (k0 > kbeg && cur.valid) {  // continue from the partial of the earlier segments
#pragma unroll
        for (int dt = 0; dt < D / 16; ++dt) {
          const bf16x4 x = *reinterpret_cast<const bf16x4 *>(a.pdq + (size_t)cur.prow * D + acc_dim(dt, quad));
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[dt][i] = (float)x[i];
        }
      }
#pragma unroll
      for (int t = 0; t < MAXT; ++t)
        if (t < nfull) bc_dq_tile<D, false>(acc, cur, kt + t * P::BYTES, vt + t * P::BYTES, ln, 32 * t, nk, sl2);
      if (nk & 31) bc_dq_tile<D, true>(acc, cur, kt + nfull * P::BYTES, vt + nfull * P::BYTES, ln, 32 * nfull, nk, sl2);
      store_partial_row<D>(a.pdq, cur.prow, acc, cur.valid);
      cur = nxt;
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
  const int32_t *row = a.idx + ((size_t)tok * a.Hkv + g) * a.T;
  int nv = 0;  // rows are ascending with the -1 padding at the end
  for (int j = 0; j < a.T; ++j) nv += row[j] >= 0 ? 1 : 0;
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
// Forward: 16-column blocks per wavefront, wavefronts per workgroup and per SIMD (see m_slc_fwd_bc for the figures).
template <int D> struct BcFwdShape { static constexpr int CB = 2, NW = 8, KSEG = 256, WPE = 4; };
template <> struct BcFwdShape<64> { static constexpr int CB = 1, NW = 8, KSEG = 256, WPE = 4; };
template <> struct BcFwdShape<128> { static constexpr int CB = 2, NW = 8, KSEG = 256, WPE = 2; };

// upper bound of the number of chunks: every (KV head, block) list adds at most one partly filled chunk
unsigned chunk_bound(const MfmaView &v, int chunk_len) {
  const size_t entries = (size_t)v.N * v.Hkv * v.T;
  return (unsigned)(entries / chunk_len + (size_t)v.Hkv * v.Ns);
}

template <int D>
int launch_slc_forward(const MfmaView &v, const bf16_t *q, const SelIndex &sel, const SlcPartials &part,
                       hipStream_t s) {
  using BS = BcFwdShape<D>;
  auto kernel = m_slc_fwd_bc<D, BS::CB, BS::NW, BS::KSEG, BS::WPE>;
  static std::once_flag once;  // raise the dynamic LDS limit once per process for this instantiation
  std::call_once(once, [&] {
    (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  });
  BcFwdArgs b{v, q, sel.list, sel.bc_chunk_start, sel.rank, sel.bc_order, part.o, part.ml};
  kernel<<<dim3((chunk_bound(v, sel.bc_chunk_len) + 7) / 8 * 8), 64 * BS::NW, bc_lds_bytes<D, BS::KSEG>(), s>>>(b);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}

template <int D>
int launch_slc_dq(const MfmaView &v, const BwdBuffers &w, hipStream_t s) {
  static std::once_flag once;
  std::call_once(once, [] {
    (void)hipFuncSetAttribute((const void *)m_bwd_dq_bc<D, DQ_WAVES, DQ_KSEG>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              160 * 1024);
  });
  const size_t NH = (size_t)v.N * v.Hq;
  BcDqArgs b{v, w.Qs, w.dOg + NH * D, w.lse2s + NH, w.deltag + NH, w.sel.list, w.sel.bc_chunk_start, w.sel.rank, w.sel.bc_order, w.part.o};
  m_bwd_dq_bc<D, DQ_WAVES, DQ_KSEG><<<dim3((chunk_bound(v, w.sel.bc_chunk_len) + 7) / 8 * 8), 64 * DQ_WAVES, bc_dq_lds_bytes<D, DQ_KSEG>(), s>>>(b);
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
                     void *out_branch, float *lse, void *out, hipStream_t s) {
  MergeArgs m{part.o, part.ml, idx, (const bf16_t *)gates, (bf16_t *)out_branch, lse, (bf16_t *)out,
              v.N, v.Hq, v.Hkv, v.hs, v.T, D};
  const size_t threads = (size_t)v.N * v.Hq * (D / 8);
  m_slc_merge<<<(unsigned)((threads + 255) / 256), 256, 0, s>>>(m);
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
