// bf16 MFMA backward kernels of SSA for gfx950.
//
// The paper states no backward pass; this is the softmax-attention gradient of eq. (2)-(4) with the selected
// index sets held constant, plus the gradient of the mean pool of eq. (5).  Per (query row, key) pair of a
// branch b with gate w_b:  P = exp(S - lse_b),  dP = <dO, V>,  dS = P (w_b dP - delta_b) scale,
// delta_b = w_b <dO, O_b>;  dV += w_b P dO,  dQ += dS K,  dK += dS Q.
//
// Three kernel families, all free of floating-point atomics (results do not depend on scheduling):
//   * m_bwd_dq: query-centric, same walk as the forward kernels (transposed scores, keys in the lanes), for the
//     compression and window branches;
//   * m_slc_bwd: the selection branch, block-centric like its forward kernel: dK, dV and one partial dQ row per selected
//     block, added per token in rank order by m_dq_merge; where long blocks dominate and at head_dim 128, two kernels, m_bwd_dq_bc and m_bwd_dkv;
//   * m_bwd_dkv (compression and window branch in one launch, with the sums of the selection branch's chunks): key-centric; a wavefront owns 16*KB keys and streams the query rows that attend to them
//     (scores with the query rows in the lanes); the contractions over query rows take Q^T and dO^T from the
//     staged row-major tiles through the transposing LDS read.
#include "mfma_common.h"
#include "cmp_form.h"
#include "mfma_launch.h"
#include "mfma_qc.h"
#include "profile.h"
#include "sel_device.h"

#include <mutex>

namespace {

// ---------------------------------------------------------------------------------------------------------
// Pre-pass: dgates, per-row scalars in sorted order, sorted copies of Q and dO.
// One workgroup per sorted token position.
// ---------------------------------------------------------------------------------------------------------
struct PreArgs {
  const bf16_t *Q, *dO, *Ob, *gates;
  const float *lse;
  const int32_t *perm;
  int N, Hq, Hkv, hs, D;
  bf16_t *dgates;               // [N,Hq,3] caller order
  float *lse2s, *deltas, *gws;  // [3][N(pos)][Hq]
  float *deltag;                // [3][N(pos)][Hq]: delta taken over the rounded gate * dO rows (see below)
  bf16_t *Qs, *dOg;             // sorted row-major copies: Q [N(pos)][Hq][D], gate_b * dO [3][N(pos)][Hq][D]
};

// BESIDE: with the index's count pass, whose own LDS a token's dO rows leave no room for where they take all there is.
template <bool BESIDE>
__global__ __launch_bounds__(256) void m_bwd_pre(PreArgs a, SelBeside sel) {
  extern __shared__ __align__(16) bf16_t tile[];  // [Hq*D]: the token's dO rows
  if constexpr (BESIDE)
    if ((int)blockIdx.x < sel.n) return sel_beside<256, true, false>(sel, blockIdx.x, tile);
  const int pos = (int)blockIdx.x - sel.n, tok = a.perm[pos];
  const int HD = a.Hq * a.D;
  const size_t base = (size_t)tok * HD;
  bf16_t *td = tile;
  // The kernels that contract over dO rows of one branch (selection dQ, all dK/dV) take gate_b * dO: with it
  // dP_b = gate_b * (dO V^T) and dV_b = P^T (gate_b * dO) carry the gate of eq. (4) without any per-row multiplication.
  for (int e = threadIdx.x * 8; e < HD; e += blockDim.x * 8) {
    const bf16x8 xq = ld8(a.Q + base + e), xd = ld8(a.dO + base + e);
    *reinterpret_cast<bf16x8 *>(td + e) = xd;
    *reinterpret_cast<bf16x8 *>(a.Qs + (size_t)pos * HD + e) = xq;
    const bf16_t *gt = a.gates + ((size_t)tok * a.Hq + e / a.D) * 3;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const float w = bf16_to_f32(gt[b]);
      bf16x8 y;
#pragma unroll
      for (int j = 0; j < 8; ++j) y[j] = (__bf16)(w * (float)xd[j]);
      *reinterpret_cast<bf16x8 *>(a.dOg + ((size_t)b * a.N + pos) * HD + e) = y;
    }
  }
  __syncthreads();
  // dgates and the row scalars: D/8 lanes per head (8 elements each), 256 / (D/8) heads per pass
  const int per = a.D / 8;  // 4, 8 or 16 lanes per head
  for (int h0 = 0; h0 < a.Hq; h0 += 256 / per) {
    const int h = h0 + threadIdx.x / per, part = threadIdx.x % per;
    // acc: <dO, O_b> (dgates, and delta_b = gate_b * it).  accg: <gate_b * dO as it was rounded into dOg, O_b>: the
    // kernels that read dOg subtract THIS delta from their dP, so that the two stay the same sum over the same numbers
    // (a softmax over one or two keys has dP = delta up to rounding, and dS = P (dP - delta) is what is left of it).
    float acc[3] = {0.f, 0.f, 0.f}, accg[3] = {0.f, 0.f, 0.f};
    if (h < a.Hq) {
      const bf16x8 go = *reinterpret_cast<const bf16x8 *>(td + h * a.D + 8 * part);
      const bf16_t *gt = a.gates + ((size_t)tok * a.Hq + h) * 3;
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const bf16x8 ob = ld8(a.Ob + (((size_t)b * a.N + tok) * a.Hq + h) * a.D + 8 * part);
        const float w = bf16_to_f32(gt[b]);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          acc[b] += (float)go[j] * (float)ob[j];
          accg[b] += (float)(__bf16)(w * (float)go[j]) * (float)ob[j];
        }
      }
    }
    for (int off = 1; off < per; off <<= 1)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        acc[b] += __shfl_xor(acc[b], off);
        accg[b] += __shfl_xor(accg[b], off);
      }
    if (h < a.Hq && part < 3) {
      const int b = part;
      const float dot = b == 0 ? acc[0] : (b == 1 ? acc[1] : acc[2]);
      const size_t th = (size_t)tok * a.Hq + h;
      const float w = bf16_to_f32(a.gates[th * 3 + b]);
      a.dgates[th * 3 + b] = f32_to_bf16(dot);
      const size_t s = ((size_t)b * a.N + pos) * a.Hq + h;
      a.lse2s[s] = a.lse[((size_t)b * a.N + tok) * a.Hq + h] * LOG2E;
      a.deltas[s] = w * dot;
      a.gws[s] = w;
      a.deltag[s] = b == 0 ? accg[0] : (b == 1 ? accg[1] : accg[2]);
    }
  }
}

// ---------------------------------------------------------------------------------------------------------
// dQ: query-centric
// ---------------------------------------------------------------------------------------------------------
struct DqArgs {
  MfmaView v;
  const bf16_t *Q, *dO;
  const float *lse2s, *deltas, *gws;  // [3][N(pos)][Hq]
  float *dQp;  // [N(pos)][Hq][D] fp32: compression + window part of dQ
};

// dS of a 32-key tile with raw scores s and dP, and dQ^T += K^T dS^T (the K rows again, read through the transposing LDS load).
// lse2 per column; gws, dls: gate and delta with the softmax scale folded in, dS = P (gate dP - delta) scale.
template <int D>
__device__ inline void dq_tile(f32x16 (&acc)[D / 32], const f32x16 &s, const f32x16 &dp, lds_cptr kt, const typename T32<D, true>::Lanes &ln,
                               float sl2, float lse2, float gws, float dls) {
#pragma unroll
  for (int kc = 0; kc < 2; ++kc) {
    bf16x8 ds;
#pragma unroll
    for (int j = 0; j < 8; ++j)
      ds[j] = (__bf16)(fast_exp2(__builtin_fmaf(s[8 * kc + j], sl2, -lse2)) * __builtin_fmaf(gws, dp[8 * kc + j], -dls));
#pragma unroll
    for (int db = 0; db < D / 32; ++db) acc[db] = mfma32(T32<D, true>::tr(kt, ln, db, kc), ds, acc[db]);
  }
}

// LDS plan of the dQ kernel (bytes): two stages (K rows, V rows)
template <int D>
__host__ __device__ inline size_t dq_lds_bytes() { return (size_t)4 * T32<D, true>::BYTES; }

// dQ of the compression branch, then of the (small) window branch, in the sorted token order; the sum is kept in fp32 by
// sorted position (dQp) for the merge with the selection branch's partials.  Bound as the forward walk (per 32 x 32 scores 384
// matrix cycles and about 280 of vector work at head_dim 64).  Three wavefronts per SIMD at head_dim 64 (163 registers).
// 62k tokens, 16 heads of 64: 1058 -> 932 us (two blocks of 16 columns per wavefront at two per SIMD before), 21k tokens in three
// 64^3 shells 140 -> 111, sequences 748 -> 640, 153k tokens, heads of 128: 8.8 -> 6.8 ms.
template <int D, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 32 ? 4 : D == 64 ? 3 : 2))) void m_bwd_dq(DqArgs a, SelBeside sel) {
  extern __shared__ __align__(16) unsigned char smem[];
  if ((int)blockIdx.x < sel.n) return sel_beside<64 * NW, false, true>(sel, blockIdx.x, smem);
  using T = T32<D, true>;
  unsigned char *stage0 = smem;
  const int h = threadIdx.x >> 5 & 1;
  const int N = a.v.N, TW = 32 * NW / a.v.hs;
  const TileMap tm = xcd_tile_map((N + TW - 1) / TW, a.v.Hkv, (int)blockIdx.x - sel.n);
  if (!tm.valid) return;
  const int g = tm.g, wg_pos0 = tm.tile * TW, wg_last = min(wg_pos0 + TW, N) - 1;
  const QCol q = query_col(a.v, wg_pos0, g);
  bf16x8 qop[D / 16], dop[D / 16];
  load_col<D>(a.Q, a.v, q, qop);
  load_col<D>(a.dO, a.v, q, dop);
  const size_t row = (size_t)q.pos * a.v.Hq + q.h;  // of the per-row arrays, which are laid out by sorted position
  const size_t NH = (size_t)N * a.v.Hq;
  f32x16 acc[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db) acc[db] = splat16(0.f);
  const float sl2 = in_vgpr(a.v.sl2), scale = a.v.scale;
  const uint32_t kstride = (uint32_t)(a.v.Hkv * D);
  const typename T::Lanes ln = T::lanes();
  // one key range per branch: the items (windows) of the workgroup's tokens are neighbours, and so are their keys
#pragma unroll 1
  for (int branch = 0; branch <= 2; branch += 2) {
    const int32_t *of_tok = branch == 0 ? a.v.tok_item : a.v.tok_win, *start = branch == 0 ? a.v.cmp_batch : a.v.win_start;
    const bf16_t *K = (branch == 0 ? a.v.Kc : a.v.Ks) + (size_t)g * D, *V = (branch == 0 ? a.v.Vc : a.v.Vs) + (size_t)g * D;
    const int r0 = uniform(of_tok[wg_pos0]), r1 = uniform(of_tok[wg_last]), own = of_tok[q.pos];
    const int rs = uniform(start[r0]), re = uniform(start[r1 + 1]), lo = start[own], hi = start[own + 1];
    const float lse2 = a.lse2s[branch * NH + row], gws = a.gws[branch * NH + row] * scale, dls = a.deltas[branch * NH + row] * scale;
    t32_pipeline<D, 2, 64 * NW, 32, false>(T32Src<2>{{K, V}, kstride}, stage0, rs, re, [&](lds_cptr kt, int kb) {
      f32x16 s = t32_scores<D, true>(qop, kt, ln, splat16(0.f)), dp = splat16(0.f);
      if (r0 != r1 || kb + 32 > re) t32_only_keys(s, kb, lo, hi);
      dp = t32_scores<D, true>(dop, kt + T::BYTES, ln, dp);
      dq_tile<D>(acc, s, dp, kt, ln, sl2, lse2, gws, dls);
    });
  }
  if (!q.valid) return;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int i = 0; i < 16; i += 4)
      *reinterpret_cast<f32x4 *>(a.dQp + row * D + 32 * db + 16 * (i >> 3) + 8 * h + (i & 4)) =
          f32x4{acc[db][i], acc[db][i + 1], acc[db][i + 2], acc[db][i + 3]};
}

// ---------------------------------------------------------------------------------------------------------
// dK/dV: key-centric
// ---------------------------------------------------------------------------------------------------------
// What a launch serves: the selection branch; or the window branch, the compression branch and the sums of the selection branch's chunks.
// The window's walks are the longest chains and too few to fill the chip, the sums wait for memory alone: beside the compression branch
// both cost next to nothing.  Three launches -> one, us: 11k tokens 140 -> 90, 21k in three shapes 212 -> 170, 62k 1420 -> 1268, 65k in
// sequences 882 -> 772.  (The sums at the end of the window's walks instead of in workgroups of their own: 5k tokens, a whole pass, 451 us
// in three launches, 472, 404.)
enum { DKV_CMP_WIN = 0, DKV_SLC = 1 };

struct DkvArgs {
  MfmaView v;
  const bf16_t *Qs, *dOg;             // sorted copies: Q [N(pos)][Hq][D], gate_b * dO [3][N(pos)][Hq][D]
  const float *lse2s, *deltag;        // [3][N(pos)][Hq]; delta over the rounded gate * dO rows
  const int32_t *sel_list;            // selection branch: query positions per (g, block)
  const int32_t *chunk_start;         // selection branch: [Hkv*Ns+1] first work chunk of each (g, block)
  const ChunkRef *chunk_order;        // selection branch: execution order of the work chunks
  const int32_t *part_row_start;      // selection branch: [Hkv*Ns+1] first row of each (g, block)'s partial sums
  const int32_t *tok_slc;             // [N(pos)] selection block
  float *dKs, *dVs;                   // [N(pos)][Hkv][D]: window branch
  float *pK, *pV;                     // [rows][D]: selection branch, partial sums per chunk
  float *dKc, *dVc;                   // [q_splits][Nc][Hkv][D]: compression branch, partial sums per part of the query range
  int slc_tiles, win_tiles, cmp_tiles;  // key tiles reserved per block (window, item) in the grid
  int n_win, n_cmp;                   // workgroups of the window and the compression branch per KV head
  int q_splits;                       // compression branch: query range split into this many parts
};

// LDS stage of the dK/dV kernels: ST tiles of 32 query rows each, of Q and of gate * dO (PTile layout: read both as
// they are and through the transposing LDS load), and two scalars per row: lse in log2 units and -delta.  The gate needs no
// scalar of its own: it rides on the dO rows, so dP = (gate dO) V^T and dV += P^T (gate dO) already carry it.
template <int D, int ST>
struct DkvStage {
  static constexpr int TILES_B = 2 * ST * PTile<D>::BYTES;  // Q tiles, then dO tiles
  static constexpr int BYTES = TILES_B + 2 * 32 * ST * 4;   // + [2][32*ST] floats
};

// The sums of a key's partial dK and dV over the chunks of its block's list, in chunk order, into the rows of the first chunk.  One thread
// per (sorted position, 4 dims) of KV head g.
template <int D, int NTHR>
__device__ inline void sum_chunks(const DkvArgs &a, int g, int wg) {
  const size_t i = (size_t)wg * NTHR + threadIdx.x;
  const int pos = (int)(i / (D / 4)), dim = (int)(i % (D / 4)) * 4;
  if (pos >= a.v.N) return;
  const int b = a.tok_slc[pos], list = g * a.v.Ns + b, b0 = a.v.slc_start[b], klen = a.v.slc_start[b + 1] - b0;
  const int chunks = a.chunk_start[list + 1] - a.chunk_start[list];
  if (chunks < 2) return;
  const size_t at = ((size_t)a.part_row_start[list] + (size_t)(pos - b0)) * D + dim, step = (size_t)klen * D;
  f32x4 sk = {0.f, 0.f, 0.f, 0.f}, sv = sk;
#pragma unroll 8
  for (int c = 0; c < chunks; ++c) {
    sk += *reinterpret_cast<const f32x4 *>(a.pK + at + c * step);
    sv += *reinterpret_cast<const f32x4 *>(a.pV + at + c * step);
  }
  *reinterpret_cast<f32x4 *>(a.pK + at) = sk;
  *reinterpret_cast<f32x4 *>(a.pV + at) = sv;
}

// A workgroup owns 16*KB*NW keys of one block (16*KB per wavefront, held in registers as MFMA B operands with their
// dK and dV accumulators) and streams the query rows that attend to them in stages of ST tiles of 32 rows (32/h_s
// token slots each), staged through LDS once per workgroup, double buffered, ONE barrier per stage: the loads of
// stage i+1 are in flight while stage i is consumed and land in the other buffer before the barrier.
template <int D, int KB, int MODE, int NW, int ST>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 32 ? 3 : 2))) void m_bwd_dkv(DkvArgs a) {
  const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, quad = lane >> 4;
  const int hs = a.v.hs, Hq = a.v.Hq;
  constexpr int WG_KEYS = 16 * KB * NW, NTHR = 64 * NW;
  using P = PTile<D>;
  using SG = DkvStage<D, ST>;
  int g, blk, tile, split = 0;
  // key range of the block and query source
  int kbeg, kend, qbeg = 0, qend = 0;
  size_t out_row0 = 0;  // selection branch: first row of this chunk's partial sums
  const bf16_t *Kr = a.v.Ks, *Vr = a.v.Vs;
  const bool win = MODE == DKV_CMP_WIN && (int)blockIdx.x < a.n_win;
  if (MODE == DKV_SLC) {
    // the key tiles of one work chunk get workgroup ids 8 apart, i.e. they run on the same XCD close in
    // time, so the chunk's query rows are fetched into that L2 once.
    const int per8 = 8 * a.slc_tiles;
    const int nkeys = a.v.Hkv * a.v.Ns, wi = (int)(blockIdx.x / per8) * 8 + (int)(blockIdx.x % 8);
    if (wi >= a.chunk_start[nkeys]) return;
    const ChunkRef cr = a.chunk_order[wi];
    const int key = cr.key;
    g = key / a.v.Ns; blk = key % a.v.Ns; tile = (int)(blockIdx.x % per8) / 8;
    kbeg = a.v.slc_start[blk]; kend = a.v.slc_start[blk + 1];
    qbeg = cr.first;
    qend = cr.first + cr.count;
    out_row0 = (size_t)a.part_row_start[key] + (size_t)cr.chunk * (kend - kbeg);
  } else if (win) {
    g = blockIdx.y; blk = (int)blockIdx.x / a.win_tiles; tile = (int)blockIdx.x % a.win_tiles;
    kbeg = a.v.win_start[blk]; kend = a.v.win_start[blk + 1];
    qbeg = kbeg; qend = kend;
  } else {
    const int w = (int)blockIdx.x - a.n_win;
    g = blockIdx.y;
    if (w >= a.n_cmp) return sum_chunks<D, NTHR>(a, g, w - a.n_cmp);
    const int per_split = a.n_cmp / a.q_splits, x = w % per_split;
    split = w / per_split;
    blk = x / a.cmp_tiles;  // batch item
    tile = x % a.cmp_tiles;
    kbeg = a.v.cmp_batch[blk]; kend = a.v.cmp_batch[blk + 1];
    const int q0 = a.v.item_start[blk], q1 = a.v.item_start[blk + 1];
    const int per = (q1 - q0 + a.q_splits - 1) / a.q_splits;
    qbeg = min(q1, q0 + split * per); qend = min(q1, qbeg + per);
    Kr = a.v.Kc; Vr = a.v.Vc;
  }
  const size_t branch_rows = (size_t)(MODE == DKV_SLC ? 1 : win ? 2 : 0) * a.v.N * Hq;
  const bf16_t *dOs = a.dOg + branch_rows * D;
  if (kbeg + tile * WG_KEYS >= kend) return;             // whole workgroup beyond the block (uniform)
  const int k0 = kbeg + tile * WG_KEYS + wid * 16 * KB;  // this wave's first key
  const bool wave_on = k0 < kend;                        // idle wavefronts still help staging and keep the barriers
  const size_t kstride = (size_t)a.v.Hkv * D;
  // B operands: this wave's keys (column n of key block kbk), all of D (rows past the block are padded: in bounds)
  bf16x8 kop[KB][D / 32], vop[KB][D / 32];
#pragma unroll
  for (int kbk = 0; kbk < KB; ++kbk) {
    const size_t off = (size_t)(k0 + 16 * kbk + n) * kstride + (size_t)g * D + 8 * quad;
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks) {
      kop[kbk][ks] = ld8(Kr + off + 32 * ks);
      vop[kbk][ks] = ld8(Vr + off + 32 * ks);
    }
  }
  f32x4 dk[KB][D / 16], dv[KB][D / 16];
#pragma unroll
  for (int kbk = 0; kbk < KB; ++kbk)
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) dk[kbk][dt] = dv[kbk][dt] = f32x4{0.f, 0.f, 0.f, 0.f};

  extern __shared__ __align__(16) unsigned char smem[];
  const int slots = 32 / hs;              // token slots per 32-row tile (hs divides 16)
  const int stage_slots = ST * slots;     // token slots per stage
  const float sl2 = a.v.sl2, scale = a.v.scale;
  const typename P::Lanes ln = P::lanes();
  // what this thread stages: NI 16-byte items of Q and of dO per stage, and (threads < 3*32*ST) one scalar
  constexpr int NI = (ST * P::ITEMS + NTHR - 1) / NTHR;
  int it_off[NI], it_slot[NI], it_col[NI];  // LDS byte offset, token slot inside the stage, element offset inside the token
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    // (when the stage has fewer items than the workgroup threads, the surplus threads repeat the last items)
    const int it = min((int)threadIdx.x + NTHR * i, ST * P::ITEMS - 1);
    const int rt = it / P::ITEMS, w = it % P::ITEMS, row = w / P::SEGS, seg = w % P::SEGS;
    it_off[i] = rt * P::BYTES + P::off(row, seg);
    it_slot[i] = rt * slots + row / hs;
    it_col[i] = (g * hs + row % hs) * D + seg * 8;
  }
  static_assert(2 * 32 * ST <= NTHR, "one scalar per thread and stage");
  const bool has_sc = threadIdx.x < 2 * 32 * ST;
  const int sc_arr = (threadIdx.x / (32 * ST)) & 1, sc_r = threadIdx.x % (32 * ST);
  const int sc_slot = (sc_r >> 5) * slots + (sc_r & 31) / hs, sc_head = g * hs + (sc_r & 31) % hs;
  const float *sc_src = (sc_arr == 0 ? a.lse2s : a.deltag) + branch_rows;
  const float sc_mul = sc_arr == 1 ? -1.0f : 1.0f;
  // sorted position of the token at list index li (-1: past the end)
  // (every load of the staging code is unconditional, with a clamped index: loads under a branch would make the
  // compiler wait for ALL outstanding loads at the next use instead of for the oldest ones)
  auto position = [&](int li) {
    const int v = MODE == DKV_SLC ? a.sel_list[min(li, qend - 1)] : li;
    return li < qend ? v : -1;
  };
  // One register set and two position sets: while stage i is consumed, the rows of stage i+1 are in flight (requested
  // right after the barrier, with the positions read during stage i-1) and the positions of stage i+2 are read.  One
  // stage of lookahead is enough because the chunks run in token order (the rows mostly come from the L2), and the
  // registers a second set would take are worth more to the tile code.  Nothing loaded is touched before the stage that
  // stores it into LDS.
  struct StageRegs { bf16x8 rq[NI], rd[NI]; float sc; bool missing; };
  struct StagePos { int it[NI], sc; };
  StageRegs regs;
  StagePos pos[2];
  auto load_positions = [&](int qb, StagePos &p) {
#pragma unroll
    for (int i = 0; i < NI; ++i) p.it[i] = position(qb + it_slot[i]);
    p.sc = position(qb + sc_slot);
  };
  auto load_stage = [&](StageRegs &r, const StagePos &p) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const uint32_t off = (uint32_t)max(p.it[i], 0) * (uint32_t)(Hq * D) + (uint32_t)it_col[i];
      r.rq[i] = ld8(a.Qs + off);
      r.rd[i] = ld8(dOs + off);
    }
    r.sc = sc_src[(uint32_t)max(p.sc, 0) * Hq + sc_head];  // (threads past the scalars load one they never store)
    r.missing = sc_arr == 0 && p.sc < 0;  // a missing row gets lse = +inf: it contributes exp2(-inf) = 0
  };
  auto store_stage = [&](const StageRegs &r, unsigned char *stage) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      *reinterpret_cast<bf16x8 *>(stage + it_off[i]) = r.rq[i];
      *reinterpret_cast<bf16x8 *>(stage + ST * P::BYTES + it_off[i]) = r.rd[i];
    }
    if (has_sc) ((float *)(stage + SG::TILES_B))[threadIdx.x] = r.missing ? INFINITY : r.sc * sc_mul;
  };

  load_positions(qbeg, pos[0]);
  load_positions(qbeg + stage_slots, pos[1]);
  load_stage(regs, pos[0]);
  int buf = 0;
  // stage qb: `regs` holds its rows; `p_rows` the positions of stage qb+1, `p_next` is refilled with those of stage qb+2
  auto do_stage = [&](int qb, const StagePos &p_rows, StagePos &p_next) {
    unsigned char *stage = smem + (size_t)buf * SG::BYTES;
    store_stage(regs, stage);
    __syncthreads();
    load_stage(regs, p_rows);                       // rows of the next stage; their positions were read one stage ago
    load_positions(qb + 2 * stage_slots, p_next);   // (past the end of the list: position -1, row 0 is loaded and dropped)
    buf ^= 1;
    if (!wave_on) return;
    const lds_cptr st0 = (lds_cptr)stage;
    const __attribute__((address_space(3))) float *scal =
        (const __attribute__((address_space(3))) float *)((lds_cptr)stage + SG::TILES_B) + 8 * quad;
#pragma unroll
    for (int rt = 0; rt < ST; ++rt) {
      // (row tiles past the end of the list are not skipped: their rows carry lse = +inf and add exact zeros, and a
      // stage without branches lets the tiles' matrix and vector work interleave)
      const lds_cptr Qt = st0 + rt * P::BYTES, Dt = st0 + (ST + rt) * P::BYTES;
      // this lane's eight consecutive query rows 8*quad .. +7 of the tile: row j is element j & 3 of sub-tile j >> 2
      float lse2[8], nd[8];  // lse (log2 units), -delta
      f32x4 s[KB][2], dp[KB][2];
      // dS = P (dP - delta) scale: the scale is applied once to the dK sums at the end.  With 32 keys per wavefront the
      // dP accumulators START from -delta of their rows, so the matrix instruction leaves dP - delta and dS costs one
      // multiplication per element; with 16 keys per wavefront (d = 128) the tile is too short to wait for the scalars
      // before its first matrix instruction, and -delta is added afterwards.
      constexpr bool DELTA_FIRST = KB > 1;
      {
        typedef const __attribute__((address_space(3))) f32x4 *f4p;
        const f32x4 l0 = *(f4p)(scal + 32 * rt), l1 = *(f4p)(scal + 32 * rt + 4);
        const f32x4 d0 = *(f4p)(scal + 32 * (ST + rt)), d1 = *(f4p)(scal + 32 * (ST + rt) + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          lse2[j] = l0[j]; lse2[4 + j] = l1[j];
          nd[j] = d0[j]; nd[4 + j] = d1[j];
        }
#pragma unroll
        for (int kbk = 0; kbk < KB; ++kbk) {
          s[kbk][0] = s[kbk][1] = f32x4{0.f, 0.f, 0.f, 0.f};
          dp[kbk][0] = DELTA_FIRST ? d0 : f32x4{0.f, 0.f, 0.f, 0.f};
          dp[kbk][1] = DELTA_FIRST ? d1 : f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
#pragma unroll
      for (int sa = 0; sa < 2; ++sa)
#pragma unroll
        for (int ks = 0; ks < D / 32; ++ks) {
          const bf16x8 qa = p_row_operand<D>(Qt, ln, sa, ks), da = p_row_operand<D>(Dt, ln, sa, ks);
#pragma unroll
          for (int kbk = 0; kbk < KB; ++kbk) {
            s[kbk][sa] = mfma16(qa, kop[kbk][ks], s[kbk][sa]);
            dp[kbk][sa] = mfma16(da, vop[kbk][ks], dp[kbk][sa]);
          }
        }
      bf16x8 pw[KB], ds[KB];
#pragma unroll
      for (int kbk = 0; kbk < KB; ++kbk)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float sv = j < 4 ? s[kbk][0][j & 3] : s[kbk][1][j & 3];
          const float dpv = j < 4 ? dp[kbk][0][j & 3] : dp[kbk][1][j & 3];  // gate * dP (- delta)
          const float p = fast_exp2(__builtin_fmaf(sv, sl2, -lse2[j]));
          pw[kbk][j] = (__bf16)p;
          ds[kbk][j] = (__bf16)(p * (DELTA_FIRST ? dpv : dpv + nd[j]));
        }
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) {
        const bf16x8 qt = p_tr_operand<D>(Qt, ln, dt), dot = p_tr_operand<D>(Dt, ln, dt);
#pragma unroll
        for (int kbk = 0; kbk < KB; ++kbk) {
          dv[kbk][dt] = mfma16(dot, pw[kbk], dv[kbk][dt]);
          dk[kbk][dt] = mfma16(qt, ds[kbk], dk[kbk][dt]);
        }
      }
    }
  };
  for (int qb = qbeg; qb < qend; qb += 2 * stage_slots) {
    do_stage(qb, pos[1], pos[0]);
    do_stage(qb + stage_slots, pos[0], pos[1]);  // (may lie wholly past the end: adds exact zeros; a branch here would
                                                 // cost a wait for all outstanding loads per iteration)
  }
  if (!wave_on) return;
  // --- store: lane holds dims acc_dim(dt, quad) + i of key column n
  float *oK = MODE == DKV_SLC ? a.pK : win ? a.dKs : a.dKc, *oV = MODE == DKV_SLC ? a.pV : win ? a.dVs : a.dVc;
#pragma unroll
  for (int kbk = 0; kbk < KB; ++kbk) {
    const int key = k0 + 16 * kbk + n;
    if (key >= kend) continue;
    size_t off = ((size_t)key * a.v.Hkv + g) * D;
    if (MODE == DKV_SLC) off = (out_row0 + (size_t)(key - kbeg)) * D;
    else if (!win) off += (size_t)split * a.v.Nc * kstride;
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) {
      *reinterpret_cast<f32x4 *>(oK + off + acc_dim(dt, quad)) = dk[kbk][dt] * scale;
      *reinterpret_cast<f32x4 *>(oV + off + acc_dim(dt, quad)) = dv[kbk][dt];
    }
  }
}

// ---------------------------------------------------------------------------------------------------------
// Finish: dK[tok] = dKs[pos] + (sum over the selection branch's chunks) + (sum over query splits of dKc[c]) / count(c)  (gradient of the
// mean pool), scattered back to caller order.  One workgroup per compression block.  With dKc_out/dVc_out given (the pooled
// rows were the caller's), the summed block gradients go there instead and dK, dV keep the token-level part only.
// ---------------------------------------------------------------------------------------------------------
struct FinishArgs {
  const int32_t *perm, *cmp_start, *cmp_slc, *slc_start, *chunk_start, *part_row_start;
  int Nc, Ns, Hkv, D, splits;
  const float *dKs, *dVs, *pK, *pV, *dKc, *dVc;
  bf16_t *dK, *dV;
  float *dKc_out, *dVc_out;
};
// Bound: latency of loads that depend on few others; a thread keeps 4 dims of a row and every NT/(row/4)-th part and token, whose loads
// are in flight together.  (With a thread per dim, parts and tokens one after the other: 11k tokens 35 us for 17, 21k 48 for 29, 62k 75 for 56.)
template <int NT>
__global__ __launch_bounds__(NT) void m_bwd_finish(FinishArgs a) {
  __shared__ f32x4 part[2][NT];
  const int c = blockIdx.x, cols = a.Hkv * a.D / 4, row = 4 * cols;
  const int b = a.cmp_start[c], e = a.cmp_start[c + 1], slc = a.cmp_slc[c];
  const int per = min(cols, NT), groups = NT / per, grp = threadIdx.x / per;  // (threads past the last group have nothing to do)
  const float inv = 1.0f / (float)(e - b);
  for (int c0 = 0; c0 < cols; c0 += per) {
    const int f = 4 * (c0 + (int)threadIdx.x % per);
    const bool on = grp < groups && f < row;
    f32x4 ck = {0.f, 0.f, 0.f, 0.f}, cv = ck;
    if (on)
#pragma unroll 8
      for (int s = grp; s < a.splits; s += groups) {
        const size_t at = ((size_t)s * a.Nc + c) * row + f;
        ck += *reinterpret_cast<const f32x4 *>(a.dKc + at);
        cv += *reinterpret_cast<const f32x4 *>(a.dVc + at);
      }
    part[0][threadIdx.x] = ck;
    part[1][threadIdx.x] = cv;
    __syncthreads();
    if (on) {
      ck = cv = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int i = 0; i < groups; ++i) {
        ck += part[0][i * per + threadIdx.x % per];
        cv += part[1][i * per + threadIdx.x % per];
      }
      if (a.dKc_out) {
        if (grp == 0) {
          *reinterpret_cast<f32x4 *>(a.dKc_out + (size_t)c * row + f) = ck;
          *reinterpret_cast<f32x4 *>(a.dVc_out + (size_t)c * row + f) = cv;
        }
        ck = cv = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      ck *= inv;
      cv *= inv;
      const int list = f / a.D * a.Ns + slc;
      const bool chosen = a.chunk_start[list + 1] > a.chunk_start[list];
      const size_t first = chosen ? ((size_t)a.part_row_start[list] + (size_t)(b - a.slc_start[slc])) * a.D + f % a.D : 0;  // position b's sums
#pragma unroll 4
      for (int pos = b + grp; pos < e; pos += groups) {
        const size_t src = (size_t)pos * row + f, dst = (size_t)a.perm[pos] * row + f, at = first + (size_t)(pos - b) * a.D;
        f32x4 k = *reinterpret_cast<const f32x4 *>(a.dKs + src), v = *reinterpret_cast<const f32x4 *>(a.dVs + src);
        if (chosen) {
          k += *reinterpret_cast<const f32x4 *>(a.pK + at);
          v += *reinterpret_cast<const f32x4 *>(a.pV + at);
        }
        k += ck;
        v += cv;
        bf16x4 x, y;
#pragma unroll
        for (int i = 0; i < 4; ++i) { x[i] = (__bf16)k[i]; y[i] = (__bf16)v[i]; }
        *reinterpret_cast<bf16x4 *>(a.dK + dst) = x;
        *reinterpret_cast<bf16x4 *>(a.dV + dst) = y;
      }
    }
    __syncthreads();
  }
}

// Threads of a block's workgroup.  Where there are many blocks of few pieces (of 4 dims of a token), workgroups of one or two wavefronts hold
// more blocks at a time.  us with 64 / 128 / 256 threads, sequences of 30k tokens, blocks of 4 tokens, rows of 32, 64, 128 dims (32, 64, 128 pieces): 22 / 28
// / 55, 30 / 37 / 54, 38 / 43 / 57; 80k, blocks of 32, rows of 32 (256) 20 / 22 / 30, of 64 (512) 35 / 35 / 42, of 128 (1024) 64 / 66 / 71; 62k in a
// 128^3 shell (886) 67 / 59 / 57.  Few blocks have all workgroups in flight and wait for the sums over the parts: 500 of 16 tokens, rows of 128 13 / 10 / 9.
int finish_threads(int cols, int N, int Nc) {
  if (Nc < 768) return 256;
  const long long pieces = (long long)cols * N / Nc;
  return pieces <= 256 ? 64 : pieces <= 512 ? 128 : 256;
}

constexpr int KB_KEYS_MAX = 2;  // key blocks of 16 per wavefront in the dK/dV kernels (1 at head_dim 128: registers)
// wavefronts per workgroup there (16*KB_KEYS keys each): blocks and windows hold ~130 tokens, an item's pooled keys
// thousands, so the compression branch takes wider workgroups (fewer passes over the query rows)
template <int D> struct DkvWaves { static constexpr int N = 4; };
template <> struct DkvWaves<128> { static constexpr int N = 8; };  // 16 keys per wavefront there: 128 keys per workgroup again
// 32-row tiles of query rows per LDS stage (one barrier per stage)
template <int D> struct DkvShape { static constexpr int ST = 2; };

template <int D>
int launch_backward(const MfmaView &v, const BwdBuffers &w, const void *q, const void *gates, const void *out_branch,
                    const float *lse, const int32_t *idx, const void *dout, void *dq, void *dk, void *dv, void *dgates,
                    const ssa_blocks *blk, int B, hipStream_t s) {
  const int N = v.N, Hq = v.Hq, Hkv = v.Hkv, row = Hkv * D;
  const size_t NH = (size_t)N * Hq;
  const bool two_kernels = slc_bwd_two_kernels(blk, D, Hkv, v.T);  // selection branch
  // the selection index, beside the pre-pass and the dQ kernel where it is small
  const size_t do_rows = (size_t)Hq * D * sizeof(bf16_t);
  const bool beside = sel_beside_fits(N, Hkv, v.T, v.Ns) && do_rows + SEL_COUNT_LDS <= LDS_CU;
  const SelJob j = sel_index_job(idx, v.perm, v.slc_start, N, Hkv, v.T, v.Ns, w.sel, false, two_kernels, true, beside);
  int rc = SSA_OK;
  {
    ProfScope ps(PROF_BWD_PRE, s);
    PreArgs a{(const bf16_t *)q, (const bf16_t *)dout, (const bf16_t *)out_branch, (const bf16_t *)gates, lse, v.perm,
              N, Hq, Hkv, v.hs, D, (bf16_t *)dgates, w.lse2s, w.deltas, w.gws, w.deltag, w.Qs, w.dOg};
    const SelBeside sel = beside ? sel_pass(j, SelPass::count) : sel_alone();
    const size_t sel_lds = beside ? j.lds_bytes() : 0;
    (beside ? m_bwd_pre<true> : m_bwd_pre<false>)<<<sel.n + N, 256, sel_lds > do_rows ? sel_lds : do_rows, s>>>(a, sel);
  }
  if (!beside || !j.ticket) {
    ProfScope ps(PROF_BWD_INVERT, s);
    if (!beside) rc = sel_index_count(j, s);
    if (rc == SSA_OK) rc = sel_index_scan(j, s);
    if (rc == SSA_OK && !beside) rc = sel_index_fill(j, s);
    if (rc == SSA_OK && !beside) rc = sel_index_order(j, s);  // (behind the dQ kernel its slots lie in no cache any more: 62k tokens 16.2 us for 12.4, 153k 41 for 27)
    if (rc != SSA_OK) return rc;
  }
  {
    ProfScope ps0(PROF_BWD_DQ_CMP, s);
    DqArgs a{v, (const bf16_t *)q, (const bf16_t *)dout, w.lse2s, w.deltas, w.gws, w.dQp};
    constexpr int NW0 = 4;
    const int tw0 = 32 * NW0 / v.hs;
    const SelBeside sel = beside ? sel_pass(j, SelPass::fill) : sel_alone();
    const size_t lds = dq_lds_bytes<D>(), sel_lds = beside ? j.lds_bytes() : 0;
    m_bwd_dq<D, NW0><<<dim3(sel.n + xcd_grid_size((N + tw0 - 1) / tw0, Hkv)), 64 * NW0, sel_lds > lds ? sel_lds : lds, s>>>(a, sel);
  }
  if (beside && !j.base) {
    ProfScope ps(PROF_BWD_INVERT, s, j.ticket != nullptr);
    rc = sel_index_order(j, s);
    if (rc != SSA_OK) return rc;
  }
  if (!two_kernels) {
    ProfScope ps1(PROF_BWD_SLC, s);
    rc = slc_bwd_kernel(v, D, w, blk->slc_tok_max, s);
    if (rc != SSA_OK) return rc;
  } else {
    ProfScope ps1(PROF_BWD_DQ, s);
    rc = slc_dq_kernel(v, D, w, s);
    if (rc != SSA_OK) return rc;
  }
  {
    ProfScope ps2(PROF_BWD_DQ_MERGE, s);
    rc = slc_dq_merge_kernel(v, D, w, idx, dq, s);
    if (rc != SSA_OK) return rc;
  }
  constexpr int KB_KEYS = D >= 128 ? 1 : KB_KEYS_MAX;
  constexpr int DKV_WAVES = DkvWaves<D>::N, WG_KEYS = 16 * KB_KEYS * DKV_WAVES;
  static_assert(WG_KEYS <= SSA_KEY_PAD, "key tiles may read up to WG_KEYS rows past a block");
  constexpr int ST = DkvShape<D>::ST;
  const size_t dkv_lds = (size_t)2 * DkvStage<D, ST>::BYTES;
  static std::once_flag dkv_once;
  std::call_once(dkv_once, [] {
    (void)hipFuncSetAttribute((const void *)m_bwd_dkv<D, KB_KEYS, DKV_SLC, DKV_WAVES, ST>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    (void)hipFuncSetAttribute((const void *)m_bwd_dkv<D, KB_KEYS, DKV_CMP_WIN, DKV_WAVES, ST>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  });
  DkvArgs a{v, w.Qs, w.dOg, w.lse2s, w.deltag, w.sel.list, w.sel.chunk_start, w.sel.order, w.sel.part_row_start, blk->tok_slc, w.dKs, w.dVs,
            w.pK, w.pV, w.dKc, w.dVc, (blk->slc_tok_max + WG_KEYS - 1) / WG_KEYS, (blk->win_tok_max + WG_KEYS - 1) / WG_KEYS,
            (blk->c_max + WG_KEYS - 1) / WG_KEYS, 0, 0, w.q_splits};
  if (two_kernels) {
    ProfScope ps(PROF_BWD_DKV_SLC, s);
    m_bwd_dkv<D, KB_KEYS, DKV_SLC, DKV_WAVES, ST><<<dim3((w.max_chunks + 7) / 8 * 8 * a.slc_tiles), 64 * DKV_WAVES, dkv_lds, s>>>(a);
  }
  {
    ProfScope ps(PROF_BWD_DKV_CMP_WIN, s);
    constexpr int NTHR = 64 * DKV_WAVES;
    a.n_win = blk->Nw * a.win_tiles;
    a.n_cmp = B * a.cmp_tiles * w.q_splits;
    const unsigned n_sum = (unsigned)(((size_t)N * (D / 4) + NTHR - 1) / NTHR);
    m_bwd_dkv<D, KB_KEYS, DKV_CMP_WIN, DKV_WAVES, ST><<<dim3(a.n_win + a.n_cmp + n_sum, Hkv), NTHR, dkv_lds, s>>>(a);
  }
  {
    ProfScope ps(PROF_BWD_FINISH, s);
    const FinishArgs f{v.perm, v.cmp_start, v.cmp_slc, v.slc_start, w.sel.chunk_start, w.sel.part_row_start, v.Nc, v.Ns, Hkv, D, w.q_splits,
                       w.dKs, w.dVs, w.pK, w.pV, w.dKc, w.dVc, (bf16_t *)dk, (bf16_t *)dv, w.dKc_out, w.dVc_out};
    const int nt = finish_threads(row / 4, N, v.Nc);
    (nt == 64 ? m_bwd_finish<64> : nt == 128 ? m_bwd_finish<128> : m_bwd_finish<256>)<<<v.Nc, nt, 0, s>>>(f);
  }
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}

}  // namespace

int mfma_backward_kernels(const MfmaView &v, int D, const BwdBuffers &w, const void *q, const void *gates,
                          const void *out_branch, const float *lse, const int32_t *idx, const void *dout, void *dq,
                          void *dk, void *dv, void *dgates, const ssa_blocks *blk, int B, hipStream_t s) {
  switch (D) {
    case 32: return launch_backward<32>(v, w, q, gates, out_branch, lse, idx, dout, dq, dk, dv, dgates, blk, B, s);
    case 64: return launch_backward<64>(v, w, q, gates, out_branch, lse, idx, dout, dq, dk, dv, dgates, blk, B, s);
    case 128: return launch_backward<128>(v, w, q, gates, out_branch, lse, idx, dout, dq, dk, dv, dgates, blk, B, s);
    default: return SSA_ERR_UNSUPPORTED;
  }
}
