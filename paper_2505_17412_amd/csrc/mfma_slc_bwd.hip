// Backward of the selection branch of SSA on bf16 MFMA for gfx950, in one pass: dK, dV and the partial dQ of every (block,
// token) pair.  Per (query row, key) pair: P = exp(S - lse), dS = P (dP - delta) with dP and delta already carrying the gate
// (the dO rows are gate * dO); dV += P^T dO, dK += dS^T Q, dQ += dS K (the softmax scale is applied to the finished sums).
//
// A workgroup owns the keys of one selection block (32 per wavefront, as matrix operands in registers with their dK and dV
// accumulators; the keys of a longer block in segments) and streams the query rows of a chunk of the tokens that selected the
// block through LDS, 64 rows per stage and group of wavefronts.
// Scores and dP are formed once: the dS tiles stay in registers for dK and go to LDS, transposed for free by the layout, for
// dQ of the same rows, which the wavefronts share out by output dims.  Two separate kernels form S and dP twice, 14 matrix
// products per pair instead of 10, and fetch the query rows twice; but a segment costs a whole pass over the query rows whatever
// its length, with the dQ rows of the segment before read back, so that long blocks are left to them where there are many.
//
// One launch serves blocks of every length, so that the few workgroups that end last are those of the shortest blocks.  A block of up to
// 128 keys has two groups of four wavefronts with the same keys, each with rows of its own; a longer one has all eight by their keys, so
// that dQ of a row is complete after 256.  With a launch per length (four wavefronts for up to 128 keys, eight beyond) each ended in
// workgroups that leave most compute units idle: 62k tokens, 0.27 ms for the 5 % of the pairs in short blocks.  Where no block is longer
// than 128 keys, workgroups of four wavefronts remain, two per compute unit, which need not keep step.
//
// Bound: the pipes of a SIMD take turns; per 32 keys x 32 query rows (d = 64) 40 matrix instructions of 16 cycles, 16 exponentials and
// some 100 VALU instructions, 32 LDS operands, with two wavefronts per SIMD (registers) that pass the same phase behind one barrier.
// The dQ product, a fifth of the matrix work, was two fifths of the time while it read K^T with every step and waited for each step's
// operands by themselves: K^T stays in registers now and the operands of two to four steps are requested together.  us of this kernel,
// before -> now on one card: 65k tokens in sequences, top-8, blocks of 128 keys 1017 -> 975, 192 1768 -> 1613, 256 2044 -> 1810 (760
// TFLOP/s); 62k tokens of a 128^3 shell, top-16, 3550 -> 3243; four such shapes (147k) 7337 -> 6890; sequences with blocks of 64 1476 ->
// 1400; 11k tokens of a 64^3 shell 385 -> 300.
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
};

// Geometry of a workgroup of NW wavefronts in RG groups.  Every group holds the same keys and takes its own rows of a stage; dK and dV
// of the groups are added at the end.
template <int D, int NW, int RG>
struct SlcBwdShape {
  static constexpr int GW = NW / RG;          // wavefronts per group
  static constexpr int KB = 2, ST = 2, ROWS = 32 * ST, KEYS = 16 * KB * GW, NTHR = 64 * NW;
  static constexpr int TILES = ST * RG, ALL_ROWS = ROWS * RG;  // of a stage
  static constexpr int NT = D / 16;           // output dim blocks of dQ
  static constexpr int G = GW / NT;           // wavefronts of a group that share its rows
  static constexpr int QB = ROWS / 16 / G;    // 16-row blocks per wavefront in the dQ product
  static constexpr int KS = KEYS / 32;        // contraction steps of the dQ product
  // 256 keys: dS and dQ tiles are double-buffered and the dQ product of a stage runs beside the scores of the next one, one
  // barrier per stage; 128 keys: single tiles, the product follows the scores of its own stage behind a second barrier.
  static constexpr bool DOUBLE = GW == 8;
  static constexpr int BUFS = DOUBLE ? 2 : 1, LAG = DOUBLE ? 1 : 0;
  // LDS (bytes): stages | dS tiles [BUFS][RG][KEYS][ROWS] (before the first stage the segment's K rows) | dQ tiles [BUFS][ALL_ROWS][D] |
  // partial rows [4][ALL_ROWS] | spare.  The groups' dK and dV meet where the stages were.
  static constexpr int STAGE_B = 2 * TILES * PTile<D>::BYTES + 2 * ALL_ROWS * 4;
  static constexpr int DS_GROUP_B = KEYS * ROWS * 2, DS_B = RG * DS_GROUP_B, DQ_B = ALL_ROWS * D * 2;
  static constexpr int DS_OFF = 2 * STAGE_B, DQ_OFF = DS_OFF + BUFS * DS_B, ROW_OFF = DQ_OFF + BUFS * DQ_B;
  static constexpr int SPARE = ROW_OFF + 4 * ALL_ROWS * 4, LDS_B = SPARE + 16, KT_OFF = DS_OFF;
  static_assert(GW % NT == 0 && QB >= 1, "the dQ product is shared out evenly");
  static_assert(KS * PTile<D>::BYTES <= BUFS * DS_B && (RG == 1 || 2 * KEYS * D * 4 <= 2 * STAGE_B), "the LDS plan has room");
};

// dS tile in LDS: one 128-byte row of 64 query rows per key, its eight 16-byte units (8 query rows each) permuted by the key:
// bits 1 and 2 of the permutation spread the four keys x 16 query rows that two quads of a transposing read touch over all
// banks, bits 0 and 1 the eight keys that eight lanes of a 16-byte write touch.
__device__ inline int ds_off(int key, int unit) {
  return key * 128 + ((unit ^ (((key >> 2) & 1) | (key & 2) | ((key >> 1) & 4))) << 4);
}

// A chunk of the list of one selection block.  SEG: blocks of more than KEYS keys are served.
template <int D, int NW, int RG, bool SEG>
__device__ __forceinline__ void slc_bwd_chunk(const SlcBwdArgs &a, unsigned char *smem, const ChunkRef &cr, int g, int kbeg, int kend) {
  using P = PTile<D>;
  using SH = SlcBwdShape<D, NW, RG>;
  constexpr int KB = SH::KB, ST = SH::ST, ROWS = SH::ROWS, ALL_ROWS = SH::ALL_ROWS, TILES = SH::TILES, NTHR = SH::NTHR, GW = SH::GW, QB = SH::QB, KS = SH::KS;
  const int wid = uniform((threadIdx.x >> 6) % GW), grp = RG == 1 ? 0 : uniform((threadIdx.x >> 6) / GW), lane = threadIdx.x & 63, n = lane & 15, quad = lane >> 4;
  const int hs = a.v.hs, hs_log = 31 - __builtin_clz(hs), Hq = a.v.Hq, Hkv = a.v.Hkv;  // (hs is 1, 2, 4, 8 or 16)
  const int qbeg = cr.first, qend = cr.first + cr.count;
  const size_t out_row0 = (size_t)a.part_row_start[cr.key] + (size_t)cr.chunk * (kend - kbeg);
  const size_t kstride = (size_t)Hkv * D;
  const float sl2 = a.v.sl2, scale = a.v.scale;
  const typename P::Lanes ln = P::lanes();
  const int slots = ALL_ROWS >> hs_log;  // tokens per stage
  const int n_st = (cr.count + slots - 1) / slots;

  // partial rows: ((pos*Hkv + g)*T + rank)*hs + head; the row behind the last one takes what belongs to no token
  const uint32_t dummy = (uint32_t)((size_t)a.v.N * Hq * a.v.T);

  // what this thread stages: NI 16-byte items of Q and of dO per stage, one row scalar, and (threads < slots) one token's
  // first partial row
  // (a thread's items are the same piece of rows in tiles IT_TILES apart; threads past the end repeat an item)
  static_assert(NTHR % P::ITEMS == 0, "whole tiles at a time");
  constexpr int NI = (TILES * P::ITEMS + NTHR - 1) / NTHR, IT_TILES = NTHR / P::ITEMS;
  const int it_tile = threadIdx.x / P::ITEMS % TILES;
  const int it_row = threadIdx.x % P::ITEMS / P::SEGS, it_seg = threadIdx.x % P::SEGS;
  const int it_off = it_tile * P::BYTES + P::off(it_row, it_seg);
  const int it_slot = (it_tile * 32 + it_row) >> hs_log, it_step = IT_TILES * 32 >> hs_log;
  const int it_col = (g * hs + (it_row & (hs - 1))) * D + it_seg * 8;
  const bool has_sc = threadIdx.x < 2 * ALL_ROWS;
  const int sc_arr = (threadIdx.x / ALL_ROWS) & 1, sc_r = threadIdx.x % ALL_ROWS;
  const int sc_slot = sc_r >> hs_log, sc_head = g * hs + (sc_r & (hs - 1));
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
      *reinterpret_cast<bf16x8 *>(stage + TILES * P::BYTES + it_off + i * IT_TILES * P::BYTES) = r.rd[i];
    }
    // (written by every thread, those without a scalar or a token into a spare word: a branch here would make the compiler
    // wait for everything outstanding, the stores of the dQ rows included)
    ((float *)(smem))[has_sc ? (int)((st & 1) * SH::STAGE_B + 2 * TILES * P::BYTES) / 4 + (int)threadIdx.x : SH::SPARE / 4] =
        r.missing ? INFINITY : r.sc * sc_mul;
    ((uint32_t *)(smem))[(int)threadIdx.x < slots ? SH::ROW_OFF / 4 + (st & 3) * ALL_ROWS + (int)threadIdx.x : SH::SPARE / 4] =
        qbeg + st * slots + (int)threadIdx.x < qend ? (((uint32_t)r.tok * Hkv + g) * a.v.T + r.rank) * hs : dummy;
  };

  // blocks longer than a workgroup's keys are taken in segments, dQ continuing from the partial rows of the segment before
  int ks0 = kbeg;
  do {
    const int nk = min(SH::KEYS, kend - ks0), n_ks = (nk + 31) >> 5;
    // this wavefront's tiles of 16 keys: number wid and, if there are so many, wid + GW.  Wavefronts without a tile still
    // stage rows, share the dQ product and keep the barriers.
    const int n_tiles = (nk + 15) >> 4, my_tiles = (n_tiles > wid) + (n_tiles > wid + GW);
    const int k0 = ks0 + wid * 16;
    load_positions(0, pos);
    for (int i = threadIdx.x; i < 4 * ALL_ROWS; i += NTHR) ((uint32_t *)(smem + SH::ROW_OFF))[i] = dummy;
    // K rows of the segment into LDS, zeros past its end, for the K^T operands of dQ
    constexpr int KT0 = SH::KT_OFF;
    for (int it = threadIdx.x; it < KS * P::ITEMS; it += NTHR) {
      const int t = it / P::ITEMS, w = it % P::ITEMS, row = w / P::SEGS, seg = w % P::SEGS, key = 32 * t + row;
      const bf16x8 x = key < nk ? ld8(a.v.Ks + (size_t)(ks0 + key) * kstride + (size_t)g * D + seg * 8) : zero8();
      *reinterpret_cast<bf16x8 *>(smem + KT0 + t * P::BYTES + P::off(row, seg)) = x;
    }
    bf16x8 kop[KB][D / 32], vop[KB][D / 32];  // this wavefront's keys (rows past the block are padded: in bounds)
#pragma unroll
    for (int kbk = 0; kbk < KB; ++kbk) {
      const size_t off = (size_t)min(k0 + 16 * GW * kbk + n, a.v.N + SSA_KEY_PAD / 2) * kstride + (size_t)g * D + 8 * quad;
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
    // K^T of this wavefront's dims, for the whole segment (read with every step instead, 6 LDS reads per pair of matrix instructions)
    const int kt_l = P::slot_off(4 * quad + (n >> 2), P::tr_seg(dtw) + ((n & 3) >> 1) * 2) + (n & 1) * 8;
    typedef __attribute__((address_space(3))) s16x4 *tr_ptr;
    typedef __attribute__((ext_vector_type(8))) short s16x8;
    auto tr_pair = [](lds_cptr lo_at, lds_cptr hi_at) {
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)lo_at), hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)hi_at);
      const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      return __builtin_bit_cast(bf16x8, both);
    };
    bf16x8 kt[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const lds_cptr kb = (lds_cptr)(smem + KT0) + kt_l + ks * P::BYTES;
      kt[ks] = tr_pair(kb, kb + 256);
    }
    __syncthreads();  // (the dS tiles take their place)
    // the dQ product also reads tiles that no wavefront has, up to a multiple of four
    for (int t = n_tiles; t < ((n_tiles + 3) & ~3); ++t)
      for (int i = threadIdx.x; i < SH::BUFS * RG * 128; i += NTHR)
        *reinterpret_cast<bf16x8 *>(smem + SH::DS_OFF + (i >> 7) * SH::DS_GROUP_B + t * 2048 + (i & 127) * 16) = zero8();
    f32x4 dk[KB][D / 16], dv[KB][D / 16];
#pragma unroll
    for (int kbk = 0; kbk < KB; ++kbk)
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) dk[kbk][dt] = dv[kbk][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    // lane parts of the dS and dQ tile addresses
    // (further units of a row are the first one's with bits 4..6 flipped, further tiles a constant away)
    static_assert(SH::DS_OFF % 128 == 0, "rows of the dS tile start on a multiple of their length");
    const int ds_w0 = SH::DS_OFF + grp * SH::DS_GROUP_B + ds_off(wid * 16 + n, quad);
    int ds_r0[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)  // query rows 4*(n & 3) .. +3 of the block, keys 8*quad + 4*h + (n >> 2)
      ds_r0[h] = SH::DS_OFF + grp * SH::DS_GROUP_B + ds_off(8 * quad + 4 * h + (n >> 2), 2 * qb0 + ((n >> 1) & 1)) + 8 * (n & 1);
    const int dq_w = SH::DQ_OFF + (ROWS * grp + 16 * qb0 + n) * (D * 2) + ((((acc_dim(dtw, quad) >> 3) ^ (n >> 1)) & (D / 8 - 1)) << 4) + (quad & 1) * 8;

    auto scores = [&](int st, auto tiles) {  // stage st: S, dP, P, dS; dV, dK; dS to LDS
      constexpr int KT = decltype(tiles)::value;
      unsigned char *stage = smem + (st & 1) * SH::STAGE_B;
      const lds_cptr st0 = (lds_cptr)stage + grp * ST * P::BYTES;
      const __attribute__((address_space(3))) float *scal =
          (const __attribute__((address_space(3))) float *)((lds_cptr)stage + 2 * TILES * P::BYTES) + grp * ROWS + 8 * quad;
#pragma unroll
      for (int rt = 0; rt < ST; ++rt) {
        // (kept apart here and below: operands of different steps in flight together spill, 3310 -> 3240 us)
        __builtin_amdgcn_sched_barrier(0);
        const lds_cptr Qt = st0 + rt * P::BYTES, Dt = st0 + (TILES + rt) * P::BYTES;
        float lse2[8];
        f32x4 s[KT][2], dp[KT][2];
        {
          typedef const __attribute__((address_space(3))) f32x4 *f4p;
          const f32x4 l0 = *(f4p)(scal + 32 * rt), l1 = *(f4p)(scal + 32 * rt + 4);
          const f32x4 d0 = *(f4p)(scal + ALL_ROWS + 32 * rt), d1 = *(f4p)(scal + ALL_ROWS + 32 * rt + 4);
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
          if (k0 + 16 * (GW * kbk + 1) > kend && k0 + 16 * GW * kbk + n >= kend) ds[kbk] = zero8();
          *reinterpret_cast<bf16x8 *>(smem + (SH::DOUBLE ? (st & 1) * SH::DS_B : 0) + GW * 2048 * kbk + (ds_w0 ^ (rt << 6))) = ds[kbk];
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
    // L1); rows that do not exist read the spare row, and their sums go back there.  (Requested where they are needed: a stage earlier
    // they take registers that the scores have not got.)
    struct Partials { uint64_t w[QB]; };
    auto load_partials = [&](int st, Partials &p) {
      const uint32_t *rows = (const uint32_t *)(smem + SH::ROW_OFF) + (st & 3) * ALL_ROWS;
#pragma unroll
      for (int q = 0; q < QB; ++q) {
        const int row = ROWS * grp + 16 * (qb0 + q) + n;
        const uint32_t pr = rows[row >> hs_log];
        p.w[q] = __hip_atomic_load((const uint64_t *)(a.pdq + (size_t)(pr + (pr == dummy ? 0 : row & (hs - 1))) * D + acc_dim(dtw, quad)),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    };
    const bool cont = SEG && ks0 != kbeg;
    auto dq_product = [&](int st) {  // rows of stage st: this wavefront's dims of dQ, to LDS
      Partials p{};
      if (cont) load_partials(st, p);
      f32x4 acc[QB];
#pragma unroll
      for (int q = 0; q < QB; ++q) {
        const bf16x4 x = __builtin_bit_cast(bf16x4, p.w[q]);  // (zeros in a block's first segment)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[q][i] = SEG ? (float)x[i] : 0.f;
      }
      const lds_cptr base = (lds_cptr)smem + (SH::DOUBLE ? (st & 1) * SH::DS_B : 0);
      // the operands of a few steps are requested together, the steps of tiles that the segment has not got left out in pairs
      auto steps = [&](auto from, auto to) {
        constexpr int F = decltype(from)::value, T = decltype(to)::value;
        bf16x8 op[T > F ? T - F : 1][QB];
#pragma unroll
        for (int ks = F; ks < T; ++ks)
#pragma unroll
          for (int q = 0; q < QB; ++q) op[ks - F][q] = tr_pair(base + (ds_r0[0] ^ (q << 5)) + ks * 4096, base + (ds_r0[1] ^ (q << 5)) + ks * 4096);
#pragma unroll
        for (int ks = F; ks < T; ++ks)
#pragma unroll
          for (int q = 0; q < QB; ++q) acc[q] = mfma16(kt[ks], op[ks - F][q], acc[q]);
      };
      typedef std::integral_constant<int, 0> I0;
      typedef std::integral_constant<int, 2> I2;
      typedef std::integral_constant<int, 4> I4;
      typedef std::integral_constant<int, KS - 2> L2;
      typedef std::integral_constant<int, KS> L0;
      if (KS == 4 || n_ks <= 4) {
        steps(I0(), I2());
        if (n_ks > 2) steps(I2(), I4());
      } else {
        steps(I0(), I4());
        steps(I4(), L2());
        if (n_ks > 6) steps(L2(), L0());
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
      const uint32_t *rows = (const uint32_t *)(smem + SH::ROW_OFF) + (st & 3) * ALL_ROWS;
      constexpr int CH = D / 8, ITEMS = ALL_ROWS * CH;
#pragma unroll
      for (int i0 = 0; i0 < ITEMS; i0 += NTHR) {
        const int it = i0 + (int)threadIdx.x;
        if (ITEMS % NTHR != 0 && it >= ITEMS) break;
        const int row = it / CH, ch = it % CH;
        const uint32_t pr = rows[row >> hs_log];
        const bf16x8 x = *reinterpret_cast<const bf16x8 *>(smem + SH::DQ_OFF + (SH::DOUBLE ? (st & 1) * SH::DQ_B : 0) + row * (D * 2) + (((ch ^ (row >> 1)) & (CH - 1)) << 4));
        // (unconditional: rows that do not exist go to the spare row, so that the compiler can count the stores)
        __builtin_nontemporal_store(x, reinterpret_cast<bf16x8 *>(a.pdq + (size_t)(pr + (pr == dummy ? 0 : row & (hs - 1))) * D + ch * 8));
      }
    };

    // Iteration i: rows of stage i into LDS | barrier | loads of stage i+1; finished dQ rows of the stage LAG+1 before out;
    // scores of stage i; dQ product of stage i - LAG.  Loads and stores are issued in every iteration, in this order and
    // under no condition, so that the wait for the loads at the next iteration's start leaves the younger stores in flight.
    store_dq(-1);  // (to the spare row: the loop is entered with the same loads and stores outstanding as an iteration leaves)
#pragma unroll 1
    for (int i = 0; i < n_st + 1 + SH::LAG; ++i) {
      store_stage(i, regs);
      __syncthreads();
      load_stage(i + 1, regs, pos);
      load_positions(i + 2, pos);
      store_dq(i - 1 - SH::LAG);
      if (i < n_st) {
        if (my_tiles == 2) scores(i, std::integral_constant<int, 2>());
        else if (my_tiles == 1) scores(i, std::integral_constant<int, 1>());
      }
      if (!SH::DOUBLE) __syncthreads();
      if (i >= SH::LAG && i < n_st + SH::LAG) dq_product(i - SH::LAG);
    }
    if constexpr (RG == 2) {  // dK and dV of the second group to the first
      __syncthreads();
      f32x4 *meet = reinterpret_cast<f32x4 *>(smem) + (threadIdx.x % (64 * GW));
      auto each = [&](auto what) {
#pragma unroll
        for (int kbk = 0; kbk < KB; ++kbk)
#pragma unroll
          for (int dt = 0; dt < D / 16; ++dt) {
            what(dk[kbk][dt], meet[(2 * (kbk * (D / 16) + dt)) * 64 * GW]);
            what(dv[kbk][dt], meet[(2 * (kbk * (D / 16) + dt) + 1) * 64 * GW]);
          }
      };
      if (grp == 1) each([](f32x4 &x, f32x4 &m) { m = x; });
      __syncthreads();
      if (grp == 1) return;
      each([](f32x4 &x, f32x4 &m) { x += m; });
    }
    {
#pragma unroll
      for (int kbk = 0; kbk < KB; ++kbk) {
        const int key = k0 + 16 * GW * kbk + n;
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

// NW = 4: no block has more than 128 keys; NW = 8: SEG, some have more than 256.
// Registers for two wavefronts per SIMD; at head_dim 32 and NW = 4 for three (168; two -> three, us, 32 heads of 32, top-16, blocks of 32, 64
// and 128 keys: 12k tokens 317 -> 251, 347 -> 288, 436 -> 391; 40k 939 -> 722, 1011 -> 820, 1354 -> 1228).
template <int D, int NW, bool SEG>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 32 && NW == 4 ? 3 : 2))) void m_slc_bwd(SlcBwdArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int wi = blockIdx.x;
  if (wi >= a.chunk_start[a.v.Hkv * a.v.Ns]) return;
  const ChunkRef cr = a.chunk_order[wi];
  const int g = cr.key / a.v.Ns, blk = cr.key % a.v.Ns;
  const int kbeg = a.v.slc_start[blk], kend = a.v.slc_start[blk + 1];
  if constexpr (NW == 4) slc_bwd_chunk<D, 4, 1, false>(a, smem, cr, g, kbeg, kend);
  else if (uniform(kend - kbeg) > SlcBwdShape<D, 8, 2>::KEYS) slc_bwd_chunk<D, 8, 1, SEG>(a, smem, cr, g, kbeg, kend);
  else slc_bwd_chunk<D, 8, 2, false>(a, smem, cr, g, kbeg, kend);
}

template <int D, int NW, bool SEG>
void launch(const SlcBwdArgs &a, unsigned chunks, hipStream_t s) {
  constexpr int L1 = SlcBwdShape<D, NW, 1>::LDS_B, L2 = SlcBwdShape<D, 8, 2>::LDS_B, LDS_B = NW == 8 && L2 > L1 ? L2 : L1;
  static std::once_flag once;  // raise the dynamic LDS limit once per process for this instantiation
  std::call_once(once, [] { (void)hipFuncSetAttribute((const void *)m_slc_bwd<D, NW, SEG>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_B); });
  m_slc_bwd<D, NW, SEG><<<dim3(chunks), 64 * NW, LDS_B, s>>>(a);
}

template <int D>
int launch_slc_bwd(const MfmaView &v, const BwdBuffers &w, int slc_tok_max, hipStream_t s) {
  const size_t NH = (size_t)v.N * v.Hq;
  const SlcBwdArgs a{v, w.Qs, w.dOg + NH * D, w.lse2s + NH, w.deltag + NH, w.sel.list, w.sel.chunk_start, w.sel.part_row_start, w.sel.rank,
                     w.sel.order, w.part.o, w.pK, w.pV};
  const unsigned chunks = (unsigned)w.max_chunks;
  if (slc_tok_max <= SlcBwdShape<D, 4, 1>::KEYS) launch<D, 4, false>(a, chunks, s);
  else if (slc_tok_max <= SlcBwdShape<D, 8, 1>::KEYS) launch<D, 8, false>(a, chunks, s);
  else launch<D, 8, true>(a, chunks, s);
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
