// Backward of the selection branch of SSA on bf16 MFMA for gfx950, in one pass: dK, dV and the partial dQ of every (block,
// token) pair.  Per (query row, key) pair: P = exp(S - lse), dS = P (dP - delta) with dP and delta already carrying the gate
// (the dO rows are gate * dO); dV += P^T dO, dK += dS^T Q, dQ += dS K (the softmax scale is applied to the finished sums).
//
// A workgroup owns the keys of one selection block (32 per wavefront, as matrix operands in registers with their dK and dV
// accumulators; the keys of a longer block in segments) and streams the query rows of a chunk of the tokens that selected the
// block, 64 rows per stage through LDS.
// Scores and dP are formed once: the dS tiles stay in registers for dK and go to LDS, transposed for free by the layout, for
// dQ of the same rows, which the wavefronts share out by output dims.  Two separate kernels form S and dP twice, 14 matrix
// products per pair instead of 10, and fetch the query rows twice; but a segment costs a whole pass over the query rows whatever
// its length, with the dQ rows of the segment before read back, so that long blocks are left to them where there are many.
//
// The pipes of a SIMD take turns: per 32 keys x 32 query rows (d = 64) 32 + 8 matrix instructions of 16.8 cycles (S, dP, dV, dK;
// dQ), 16 exponentials and some 100 VALU instructions, 34 LDS operands of 9 to 16 cycles, about 1430 cycles one after the other;
// 1450 are measured, with two wavefronts per SIMD (registers).  That describes the schedule and is no lower bound: all wavefronts
// pass the same phase behind one barrier, wait 41 % of their life and keep the matrix pipes 26 % busy.  Besides, a block that
// does not fill its workgroup's tiles leaves wavefronts idle.  Time of the two kernels -> one pass: 62 k tokens of a 128^3 shell
// 3344 -> 3240 us, four such shapes (147 k) 8834 -> 7200, 65 k tokens in sequences with blocks of 64 2155 -> 1300, 21 k tokens in three 64^3 shells 642 -> 506.
#include "mfma_common.h"
#include "mfma_launch.h"
#include "mfma_qc.h"

#include <mutex>

namespace {

struct SlcBwdArgs {
  MfmaView v;
  const bf16_t *Qs, *dOs;       // sorted copies [N(pos)][Hq][D]: Q, and the selection gate times dO
  const float *lse2s, *deltas;  // selection branch [N(pos)][Hq]; delta over the rounded gate * dO rows
  const int32_t *sel_list, *chunk_start, *part_row_start;  // lists of sorted positions
  const uint8_t *sel_rank;
  const ChunkRef *chunk_order;
  bf16_t *pdq;                  // [N(pos)][Hkv][T][hs][D] partial dQ, and one spare row
  float *pK, *pV;               // [rows][D] partial dK, dV per chunk
  int len_lo, len_hi;           // this launch serves the blocks of len_lo < keys <= len_hi
};

// Geometry of a workgroup of NW wavefronts.
template <int D, int NW>
struct SlcBwdShape {
  static constexpr int KB = 2, ST = 2, ROWS = 32 * ST, KEYS = 16 * KB * NW, NTHR = 64 * NW;
  static constexpr int NT = D / 16;           // output dim blocks of dQ
  static constexpr int G = NW / NT;           // groups of wavefronts that share a stage's rows
  static constexpr int QB = ROWS / 16 / G;    // 16-row blocks per wavefront in the dQ product
  static constexpr int KS = KEYS / 32;        // contraction steps of the dQ product
  // NW = 8: dS and dQ tiles are double-buffered and the dQ product of a stage runs beside the scores of the next one, one
  // barrier per stage; NW = 4: single tiles, the product follows the scores of its own stage behind a second barrier, and
  // two workgroups share a compute unit.
  static constexpr bool DOUBLE = NW == 8;
  static constexpr int BUFS = DOUBLE ? 2 : 1, LAG = DOUBLE ? 1 : 0;
  // LDS (bytes): stages | dS tiles [BUFS][KEYS][ROWS] | dQ tiles [BUFS][ROWS][D] | partial rows [4][ROWS] | spare | K tiles
  static constexpr int STAGE_B = 2 * ST * PTile<D>::BYTES + 2 * ROWS * 4;
  static constexpr int DS_B = KEYS * ROWS * 2, DQ_B = ROWS * D * 2;
  static constexpr int DS_OFF = 2 * STAGE_B, DQ_OFF = DS_OFF + BUFS * DS_B, ROW_OFF = DQ_OFF + BUFS * DQ_B;
  static constexpr int SPARE = ROW_OFF + 4 * ROWS * 4, KT_OFF = SPARE + 16;
  static constexpr int LDS_B = KT_OFF + KS * PTile<D>::BYTES;
  static_assert(NW % NT == 0 && QB >= 1, "the dQ product is shared out evenly");
};

// dS tile in LDS: one 128-byte row of 64 query rows per key, its eight 16-byte units (8 query rows each) permuted by the key:
// bits 1 and 2 of the permutation spread the four keys x 16 query rows that two quads of a transposing read touch over all
// banks, bits 0 and 1 the eight keys that eight lanes of a 16-byte write touch.
__device__ inline int ds_off(int key, int unit) {
  return key * 128 + ((unit ^ (((key >> 2) & 1) | (key & 2) | ((key >> 1) & 4))) << 4);
}

// SEG: blocks of more than KEYS keys are served, in segments (its second form of the stage loop spills 7 registers at d = 64).
template <int D, int NW, bool SEG>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void m_slc_bwd(SlcBwdArgs a) {
  using P = PTile<D>;
  using SH = SlcBwdShape<D, NW>;
  constexpr int KB = SH::KB, ST = SH::ST, ROWS = SH::ROWS, NTHR = SH::NTHR, QB = SH::QB, KS = SH::KS;
  extern __shared__ __align__(16) unsigned char smem[];
  const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, quad = lane >> 4;
  const int hs = a.v.hs, Hq = a.v.Hq, Hkv = a.v.Hkv;
  const int wi = blockIdx.x;
  if (wi >= a.chunk_start[Hkv * a.v.Ns]) return;
  const ChunkRef cr = a.chunk_order[wi];
  const int g = cr.key / a.v.Ns, blk = cr.key % a.v.Ns;
  const int kbeg = a.v.slc_start[blk], kend = a.v.slc_start[blk + 1];
  if (kend - kbeg <= a.len_lo || kend - kbeg > a.len_hi) return;
  const int qbeg = cr.first, qend = cr.first + cr.count;
  const size_t out_row0 = (size_t)a.part_row_start[cr.key] + (size_t)cr.chunk * (kend - kbeg);
  const size_t kstride = (size_t)Hkv * D;
  const float sl2 = a.v.sl2, scale = a.v.scale;
  const typename P::Lanes ln = P::lanes();
  const int slots = ROWS / hs;  // tokens per stage
  const int n_st = (cr.count + slots - 1) / slots;

  // partial rows: ((pos*Hkv + g)*T + rank)*hs + head; the row behind the last one takes what belongs to no token
  const uint32_t dummy = (uint32_t)((size_t)a.v.N * Hq * a.v.T);

  // what this thread stages: NI 16-byte items of Q and of dO per stage, one row scalar, and (threads < slots) one token's
  // first partial row
  // (a thread's items are the same piece of rows in tiles IT_TILES apart; threads past the end repeat an item)
  static_assert(NTHR % P::ITEMS == 0, "whole tiles at a time");
  constexpr int NI = (ST * P::ITEMS + NTHR - 1) / NTHR, IT_TILES = NTHR / P::ITEMS;
  const int it_tile = threadIdx.x / P::ITEMS % ST;
  const int it_row = threadIdx.x % P::ITEMS / P::SEGS, it_seg = threadIdx.x % P::SEGS;
  const int it_off = it_tile * P::BYTES + P::off(it_row, it_seg);
  const int it_slot = (it_tile * 32 + it_row) / hs, it_step = IT_TILES * 32 / hs;  // (hs is 1, 2, 4, 8 or 16)
  const int it_col = (g * hs + it_row % hs) * D + it_seg * 8;
  const bool has_sc = threadIdx.x < 2 * ROWS;
  const int sc_arr = (threadIdx.x / ROWS) & 1, sc_r = threadIdx.x % ROWS;
  const int sc_slot = sc_r / hs, sc_head = g * hs + sc_r % hs;
  const float *sc_src = sc_arr == 0 ? a.lse2s : a.deltas;
  const float sc_mul = sc_arr == 1 ? -1.0f : 1.0f;
  // (loads are unconditional with clamped indices, so the compiler's wait counts are exact)
  auto position = [&](int li) {
    const int v = a.sel_list[min(li, qend - 1)];
    return li < qend ? v : -1;
  };
  struct StageRegs { bf16x8 rq[NI], rd[NI]; float sc; bool missing; int tok, rank; };
  struct StagePos { int it[NI], sc; };
  StageRegs regs;
  StagePos pos;
  auto load_positions = [&](int st, StagePos &p) {
    const int qb = qbeg + st * slots;
#pragma unroll
    for (int i = 0; i < NI; ++i) p.it[i] = position(qb + it_slot + i * it_step);
    p.sc = position(qb + sc_slot);
  };
  auto load_stage = [&](int st, StageRegs &r, const StagePos &p) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const uint32_t off = (uint32_t)max(p.it[i], 0) * (uint32_t)(Hq * D) + (uint32_t)it_col;
      r.rq[i] = ld8(a.Qs + off);
      r.rd[i] = ld8(a.dOs + off);
    }
    r.sc = sc_src[(uint32_t)max(p.sc, 0) * Hq + sc_head];
    r.missing = sc_arr == 0 && p.sc < 0;  // a missing row gets lse = +inf: it contributes exp2(-inf) = 0
    const int lc = min(qbeg + st * slots + (int)threadIdx.x, qend - 1);
    r.tok = a.sel_list[lc];
    r.rank = a.sel_rank[lc];
  };
  auto store_stage = [&](int st, const StageRegs &r) {
    unsigned char *stage = smem + (st & 1) * SH::STAGE_B;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      *reinterpret_cast<bf16x8 *>(stage + it_off + i * IT_TILES * P::BYTES) = r.rq[i];
      *reinterpret_cast<bf16x8 *>(stage + ST * P::BYTES + it_off + i * IT_TILES * P::BYTES) = r.rd[i];
    }
    // (written by every thread, those without a scalar or a token into a spare word: a branch here would make the compiler
    // wait for everything outstanding, the stores of the dQ rows included)
    ((float *)(smem))[has_sc ? (int)((st & 1) * SH::STAGE_B + 2 * ST * P::BYTES) / 4 + (int)threadIdx.x : SH::SPARE / 4] =
        r.missing ? INFINITY : r.sc * sc_mul;
    ((uint32_t *)(smem))[(int)threadIdx.x < slots ? SH::ROW_OFF / 4 + (st & 3) * ROWS + (int)threadIdx.x : SH::SPARE / 4] =
        qbeg + st * slots + (int)threadIdx.x < qend ? (((uint32_t)r.tok * Hkv + g) * a.v.T + r.rank) * hs : dummy;
  };

  // blocks longer than a workgroup's keys are taken in segments, dQ continuing from the partial rows of the segment before
  int ks0 = kbeg;
  do {
    const int nk = min(SH::KEYS, kend - ks0), n_ks = (nk + 31) >> 5;
    // this wavefront's tiles of 16 keys: number wid and, if there are so many, wid + NW.  Wavefronts without a tile still
    // stage rows, share the dQ product and keep the barriers.
    const int n_tiles = (nk + 15) >> 4, my_tiles = (n_tiles > wid) + (n_tiles > wid + NW);
    const int k0 = ks0 + wid * 16;
    load_positions(0, pos);
    for (int i = threadIdx.x; i < 4 * ROWS; i += NTHR) ((uint32_t *)(smem + SH::ROW_OFF))[i] = dummy;
    // K rows of the segment into LDS, zeros past its end, for the K^T operands of dQ
    constexpr int KT0 = SH::KT_OFF;
    for (int it = threadIdx.x; it < KS * P::ITEMS; it += NTHR) {
      const int t = it / P::ITEMS, w = it % P::ITEMS, row = w / P::SEGS, seg = w % P::SEGS, key = 32 * t + row;
      const bf16x8 x = key < nk ? ld8(a.v.Ks + (size_t)(ks0 + key) * kstride + (size_t)g * D + seg * 8) : zero8();
      *reinterpret_cast<bf16x8 *>(smem + KT0 + t * P::BYTES + P::off(row, seg)) = x;
    }
    if (n_tiles & 1)  // the last contraction step of the dQ product also reads the tile that no wavefront has
      for (int i = threadIdx.x; i < SH::BUFS * 128; i += NTHR)
        *reinterpret_cast<bf16x8 *>(smem + SH::DS_OFF + (i >> 7) * SH::DS_B + n_tiles * 2048 + (i & 127) * 16) = zero8();
    bf16x8 kop[KB][D / 32], vop[KB][D / 32];  // this wavefront's keys (rows past the block are padded: in bounds)
#pragma unroll
    for (int kbk = 0; kbk < KB; ++kbk) {
      const size_t off = (size_t)min(k0 + 16 * NW * kbk + n, a.v.N + SSA_KEY_PAD / 2) * kstride + (size_t)g * D + 8 * quad;
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks) {
        kop[kbk][ks] = ld8(a.v.Ks + off + 32 * ks);
        vop[kbk][ks] = ld8(a.v.Vs + off + 32 * ks);
      }
    }
    load_stage(0, regs, pos);
    load_positions(1, pos);
    __syncthreads();
    const int dtw = wid % SH::NT, qb0 = wid / SH::NT * QB;  // this wavefront's share of the dQ product
    const int kt_l = P::slot_off(4 * quad + (n >> 2), P::tr_seg(dtw) + ((n & 3) >> 1) * 2) + (n & 1) * 8;
    f32x4 dk[KB][D / 16], dv[KB][D / 16];
#pragma unroll
    for (int kbk = 0; kbk < KB; ++kbk)
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) dk[kbk][dt] = dv[kbk][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    // lane parts of the dS and dQ tile addresses
    // (further units of a row are the first one's with bits 4..6 flipped, further tiles a constant away)
    static_assert(SH::DS_OFF % 128 == 0, "rows of the dS tile start on a multiple of their length");
    const int ds_w0 = SH::DS_OFF + ds_off(wid * 16 + n, quad);
    int ds_r0[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)  // query rows 4*(n & 3) .. +3 of the block, keys 8*quad + 4*h + (n >> 2)
      ds_r0[h] = SH::DS_OFF + ds_off(8 * quad + 4 * h + (n >> 2), 2 * qb0 + ((n >> 1) & 1)) + 8 * (n & 1);
    const int dq_w = SH::DQ_OFF + (16 * qb0 + n) * (D * 2) + ((((acc_dim(dtw, quad) >> 3) ^ (n >> 1)) & (D / 8 - 1)) << 4) + (quad & 1) * 8;

    auto scores = [&](int st, auto tiles) {  // stage st: S, dP, P, dS; dV, dK; dS to LDS
      constexpr int KT = decltype(tiles)::value;
      unsigned char *stage = smem + (st & 1) * SH::STAGE_B;
      const lds_cptr st0 = (lds_cptr)stage;
      const __attribute__((address_space(3))) float *scal =
          (const __attribute__((address_space(3))) float *)(st0 + 2 * ST * P::BYTES) + 8 * quad;
#pragma unroll
      for (int rt = 0; rt < ST; ++rt) {
        // (kept apart here and below: operands of different steps in flight together spill, 3310 -> 3240 us)
        __builtin_amdgcn_sched_barrier(0);
        const lds_cptr Qt = st0 + rt * P::BYTES, Dt = st0 + (ST + rt) * P::BYTES;
        float lse2[8];
        f32x4 s[KT][2], dp[KT][2];
        {
          typedef const __attribute__((address_space(3))) f32x4 *f4p;
          const f32x4 l0 = *(f4p)(scal + 32 * rt), l1 = *(f4p)(scal + 32 * rt + 4);
          const f32x4 d0 = *(f4p)(scal + ROWS + 32 * rt), d1 = *(f4p)(scal + ROWS + 32 * rt + 4);
#pragma unroll
          for (int j = 0; j < 4; ++j) { lse2[j] = l0[j]; lse2[4 + j] = l1[j]; }
#pragma unroll
          for (int kbk = 0; kbk < KT; ++kbk) {
            s[kbk][0] = s[kbk][1] = f32x4{0.f, 0.f, 0.f, 0.f};
            dp[kbk][0] = d0;  // dP starts from -delta of its row
            dp[kbk][1] = d1;
          }
        }
#pragma unroll
        for (int sa = 0; sa < 2; ++sa)
#pragma unroll
          for (int ks = 0; ks < D / 32; ++ks) {
            const bf16x8 qa = p_row_operand<D>(Qt, ln, sa, ks), da = p_row_operand<D>(Dt, ln, sa, ks);
#pragma unroll
            for (int kbk = 0; kbk < KT; ++kbk) {
              s[kbk][sa] = mfma16(qa, kop[kbk][ks], s[kbk][sa]);
              dp[kbk][sa] = mfma16(da, vop[kbk][ks], dp[kbk][sa]);
            }
          }
        __builtin_amdgcn_sched_barrier(0);
        bf16x8 pw[KT], ds[KT];
#pragma unroll
        for (int kbk = 0; kbk < KT; ++kbk) {
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const float p = fast_exp2(__builtin_fmaf(s[kbk][j >> 2][j & 3], sl2, -lse2[j]));
            pw[kbk][j] = (__bf16)p;
            ds[kbk][j] = (__bf16)(p * dp[kbk][j >> 2][j & 3]);
          }
          // keys past the block give finite or infinite garbage columns of dS that dQ must not see
          if (k0 + 16 * (NW * kbk + 1) > kend && k0 + 16 * NW * kbk + n >= kend) ds[kbk] = zero8();
          *reinterpret_cast<bf16x8 *>(smem + (SH::DOUBLE ? (st & 1) * SH::DS_B : 0) + NW * 2048 * kbk + (ds_w0 ^ (rt << 6))) = ds[kbk];
        }
#pragma unroll
        for (int dt = 0; dt < D / 16; ++dt) {
          const bf16x8 qt = p_tr_operand<D>(Qt, ln, dt), dot = p_tr_operand<D>(Dt, ln, dt);
#pragma unroll
          for (int kbk = 0; kbk < KT; ++kbk) {
            dv[kbk][dt] = mfma16(dot, pw[kbk], dv[kbk][dt]);
            dk[kbk][dt] = mfma16(qt, ds[kbk], dk[kbk][dt]);
          }
        }
      }
    };
    // this wavefront's share of the partial rows of stage st from the segment before (written by this workgroup, read past the
    // L1); rows that do not exist read the spare row, and their sums go back there
    struct Partials { uint64_t w[QB]; };
    auto load_partials = [&](int st, Partials &p) {
      const uint32_t *rows = (const uint32_t *)(smem + SH::ROW_OFF) + (st & 3) * ROWS;
#pragma unroll
      for (int q = 0; q < QB; ++q) {
        const int row = 16 * (qb0 + q) + n;
        const uint32_t pr = rows[row / hs];
        p.w[q] = __hip_atomic_load((const uint64_t *)(a.pdq + (size_t)(pr + (pr == dummy ? 0 : row % hs)) * D + acc_dim(dtw, quad)),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    };
    auto dq_product = [&](int st, auto cont, const Partials &p) {  // rows of stage st: this wavefront's dims of dQ, to LDS
      f32x4 acc[QB];
#pragma unroll
      for (int q = 0; q < QB; ++q) {
        acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (decltype(cont)::value) {
          const bf16x4 x = __builtin_bit_cast(bf16x4, p.w[q]);
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[q][i] = (float)x[i];
        }
      }
      const lds_cptr base = (lds_cptr)smem + (SH::DOUBLE ? (st & 1) * SH::DS_B : 0);
      typedef __attribute__((address_space(3))) s16x4 *tr_ptr;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        if (ks < n_ks) {
          typedef __attribute__((ext_vector_type(8))) short s16x8;
          const lds_cptr kb = (lds_cptr)(smem + KT0) + kt_l + ks * P::BYTES;
          const s16x4 klo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)kb), khi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(kb + 256));
          const s16x8 k8 = __builtin_shufflevector(klo, khi, 0, 1, 2, 3, 4, 5, 6, 7);
          const bf16x8 kt = __builtin_bit_cast(bf16x8, k8);
#pragma unroll
          for (int q = 0; q < QB; ++q) {
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(base + (ds_r0[0] ^ (q << 5)) + ks * 4096));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(base + (ds_r0[1] ^ (q << 5)) + ks * 4096));
            const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            acc[q] = mfma16(kt, __builtin_bit_cast(bf16x8, both), acc[q]);
          }
        }
#pragma unroll
      for (int q = 0; q < QB; ++q) {
        bf16x4 x;
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = (__bf16)acc[q][i];
        *reinterpret_cast<bf16x4 *>(smem + (SH::DOUBLE ? (st & 1) * SH::DQ_B : 0) + dq_w + q * 16 * D * 2) = x;
      }
    };
    auto store_dq = [&](int st) {  // the finished dQ rows of stage st go out as whole lines
      const uint32_t *rows = (const uint32_t *)(smem + SH::ROW_OFF) + (st & 3) * ROWS;
      constexpr int CH = D / 8, ITEMS = ROWS * CH;
#pragma unroll
      for (int i0 = 0; i0 < ITEMS; i0 += NTHR) {
        const int it = i0 + (int)threadIdx.x;
        if (ITEMS % NTHR != 0 && it >= ITEMS) break;
        const int row = it / CH, ch = it % CH;
        const uint32_t pr = rows[row / hs];
        const bf16x8 x = *reinterpret_cast<const bf16x8 *>(smem + SH::DQ_OFF + (SH::DOUBLE ? (st & 1) * SH::DQ_B : 0) + row * (D * 2) + (((ch ^ (row >> 1)) & (CH - 1)) << 4));
        // (unconditional: rows that do not exist go to the spare row, so that the compiler can count the stores)
        __builtin_nontemporal_store(x, reinterpret_cast<bf16x8 *>(a.pdq + (size_t)(pr + (pr == dummy ? 0 : row % hs)) * D + ch * 8));
      }
    };

    // Iteration i: rows of stage i into LDS | barrier | loads of stage i+1; finished dQ rows of the stage LAG+1 before out;
    // scores of stage i; dQ product of stage i - LAG.  Loads and stores are issued in every iteration, in this order and
    // under no condition, so that the wait for the loads at the next iteration's start leaves the younger stores in flight.
    auto stream = [&](auto cont) {
      store_dq(-1);  // (to the spare row: the loop is entered with the same loads and stores outstanding as an iteration leaves)
#pragma unroll 1
      for (int i = 0; i < n_st + 1 + SH::LAG; ++i) {
        Partials part{};
        store_stage(i, regs);
        __syncthreads();
        if constexpr (decltype(cont)::value) load_partials(i - SH::LAG, part);
        load_stage(i + 1, regs, pos);
        load_positions(i + 2, pos);
        store_dq(i - 1 - SH::LAG);
        if (i < n_st) {
          if (my_tiles == 2) scores(i, std::integral_constant<int, 2>());
          else if (my_tiles == 1) scores(i, std::integral_constant<int, 1>());
        }
        if (!SH::DOUBLE) __syncthreads();
        if (i >= SH::LAG && i < n_st + SH::LAG) dq_product(i - SH::LAG, cont, part);
      }
    };
    if (!SEG || ks0 == kbeg) stream(std::false_type());
    else if constexpr (SEG) stream(std::true_type());
    {
#pragma unroll
      for (int kbk = 0; kbk < KB; ++kbk) {
        const int key = k0 + 16 * NW * kbk + n;
        if (key >= kend) continue;
        const size_t off = (out_row0 + (size_t)(key - kbeg)) * D;
#pragma unroll
        for (int dt = 0; dt < D / 16; ++dt) {
          *reinterpret_cast<float4 *>(a.pK + off + acc_dim(dt, quad)) =
              make_float4(dk[kbk][dt][0] * scale, dk[kbk][dt][1] * scale, dk[kbk][dt][2] * scale, dk[kbk][dt][3] * scale);
          *reinterpret_cast<float4 *>(a.pV + off + acc_dim(dt, quad)) = make_float4(dv[kbk][dt][0], dv[kbk][dt][1], dv[kbk][dt][2], dv[kbk][dt][3]);
        }
      }
    }
    ks0 += SH::KEYS;
    if (SEG && ks0 < kend) {  // the next segment reads the partial rows back
      __threadfence();
      __syncthreads();
    }
  } while (SEG && ks0 < kend);
}

template <int D, int NW, bool SEG>
void launch(SlcBwdArgs a, int lo, int hi, unsigned chunks, hipStream_t s) {
  using SH = SlcBwdShape<D, NW>;
  static std::once_flag once;  // raise the dynamic LDS limit once per process for this instantiation
  std::call_once(once, [] { (void)hipFuncSetAttribute((const void *)m_slc_bwd<D, NW, SEG>, hipFuncAttributeMaxDynamicSharedMemorySize, SH::LDS_B); });
  a.len_lo = lo;
  a.len_hi = hi;
  m_slc_bwd<D, NW, SEG><<<dim3(chunks), SH::NTHR, SH::LDS_B, s>>>(a);
}

template <int D>
int launch_slc_bwd(const MfmaView &v, const BwdBuffers &w, int slc_tok_max, hipStream_t s) {
  const size_t NH = (size_t)v.N * v.Hq;
  SlcBwdArgs a{v, w.Qs, w.dOg + NH * D, w.lse2s + NH, w.deltag + NH, w.sel.list, w.sel.chunk_start, w.sel.part_row_start, w.sel.rank,
               w.sel.order, w.part.o, w.pK, w.pV, 0, 0};
  constexpr int SHORT = SlcBwdShape<D, 4>::KEYS, LONG = SlcBwdShape<D, 8>::KEYS;
  const unsigned chunks = (unsigned)w.max_chunks;
  // blocks of up to 128 keys: 4 wavefronts, two workgroups per compute unit; longer ones: 8 wavefronts, so that dQ of a
  // block is complete after 256 keys (4 wavefronts, which read the partial row of the first 128 keys back, took 3770 us for
  // 3390 with the line at 160 keys, 5170 at 192)
  launch<D, 4, false>(a, 0, SHORT, chunks, s);
  if (slc_tok_max > LONG) launch<D, 8, true>(a, SHORT, 0x7fffffff, chunks, s);
  else if (slc_tok_max > SHORT) launch<D, 8, false>(a, SHORT, LONG, chunks, s);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}

}  // namespace

int slc_bwd_kernel(const MfmaView &v, int D, const BwdBuffers &w, int slc_tok_max, hipStream_t s) {
  switch (D) {
    case 32: return launch_slc_bwd<32>(v, w, slc_tok_max, s);
    case 64: return launch_slc_bwd<64>(v, w, slc_tok_max, s);
    default: return SSA_ERR_UNSUPPORTED;
  }
}
