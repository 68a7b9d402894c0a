// 32 x 32 x 16 matrix tiles of the attention kernels (gfx950, wave64, v_mfma_f32_32x32x16_bf16): LDS tile layout, operands,
// softmax sums and row stores.
//
// Operand convention of the instruction (h = lane >> 5, n = lane & 31):
//   A (32 x 16): the lane supplies row n, contraction indices 8*h .. +7;  B (16 x 32): column n, the same indices
//   C/D (32 x 32 fp32): the lane holds column n, rows 8*(i >> 2) + 4*h + (i & 3), i = 0 .. 15
// A wavefront keeps 32 query columns and walks over tiles of 32 keys.  Scores are formed transposed (keys x queries), so that
// registers 8*kc .. +7 of a lane are, for its query, the contraction slice kc (16 keys) of the next product; the keys of a slice
// are in the order 16*kc + 8*(j >> 2) + 4*h + (j & 3), j = 0 .. 7, which the transposed operand below repeats.
//
// Why 32 columns and not 16: an operand taken from LDS (1 KB) feeds a matrix instruction of 32 cycles instead of 16.  With 16
// columns the four SIMDs of a compute unit ask for as many LDS cycles as they spend matrix cycles, and the kernels wait for LDS
// whatever their vector work is.
#pragma once

#include "mfma_common.h"

typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ inline f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
__device__ inline f32x16 splat16(float x) {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = x;
  return z;
}
// Row of register i of an accumulator tile.
__device__ inline int t32_row(int i) { return 8 * (i >> 2) + 4 * (threadIdx.x >> 5 & 1) + (i & 3); }

// A tile of 32 rows x D bf16 in LDS: D/8 planes of 512 bytes, one per 16-byte segment of a row; row r lies in slot
// r ^ swz(segment) of the plane.  Banks (16 slots of 16 bytes are all of them): a row operand reads whole planes; a transposing
// read takes 4 rows x 4 segments at a time, which bits 2, 3 of swz (the segment's low bits) spread over all banks; with SWZ bits 1
// and 0 do the same for a staging write, whose neighbouring threads hold the segments of one row.  Kernels that stage a block once
// and read it many times leave those two bits out: their lane offsets then differ between contraction steps by constants.
template <int D, bool SWZ>
struct T32 {
  static constexpr int SEGS = D / 8, BYTES = SEGS * 512, ITEMS = 32 * SEGS;
  static constexpr int NROW = SWZ ? D / 16 : 2, NTR = SWZ ? D / 32 : 1;
  __device__ static inline int swz(int seg) { return (seg & 3) << 2 | (SWZ ? (seg >> 2 & 1) << 1 | (seg >> 3 & 1) : 0); }
  __device__ static inline int off(int row, int seg) { return seg * 512 + ((row ^ swz(seg)) << 4); }
  struct Lanes {
    int row[NROW];    // row operand, contraction step ks (ks & 1 without SWZ)
    int tr[NTR][2];   // transposed operand: keys +0 .. 3 and +8 .. 11 of the slice, dim block db (the first without SWZ)
  };
  // The 32 rows of a transposed operand are the dims of block db in the order that leaves a lane with 8 consecutive dims in
  // registers 0 .. 7 (32*db + 8*h ..) and in 8 .. 15 (32*db + 16 + 8*h ..): bits 2 and 3 of row and dim change places.
  __device__ static inline Lanes lanes() {
    const int l = threadIdx.x & 63, h = l >> 5, p = l & 3, r = (l & 15) >> 2;
    Lanes x;
#pragma unroll
    for (int ks = 0; ks < NROW; ++ks) x.row[ks] = off(l & 31, 2 * ks + h);
#pragma unroll
    for (int db = 0; db < NTR; ++db)
#pragma unroll
      for (int k = 0; k < 2; ++k) x.tr[db][k] = off(4 * h + 8 * k + r, 4 * db + 2 * (l >> 4 & 1) + (p & 1)) + 8 * (p >> 1);
    return x;
  }
  typedef const __attribute__((address_space(3))) unsigned char *ptr;
  // A operand: rows of the tile, dims 16*ks + 8*h .. +7
  __device__ static inline bf16x8 row(ptr tile, const Lanes &x, int ks) {
    const int o = SWZ ? x.row[ks % NROW] : x.row[ks & 1] + (ks >> 1) * 2048;
    return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8 *>(tile + o);
  }
  // A operand: dims of block db, contraction over the keys of slice kc (ds_read_b64_tr_b16: of a group of 16 lanes lane 4*r + p
  // hands in the address of 4 dims of row r, and lane i receives dim i of the four rows)
  __device__ static inline bf16x8 tr(ptr tile, const Lanes &x, int db, int kc) {
    typedef __attribute__((ext_vector_type(4))) short s16x4;
    typedef __attribute__((ext_vector_type(8))) short s16x8;
    typedef __attribute__((address_space(3))) s16x4 *tr_ptr;
    const int add = (SWZ ? 0 : db * 2048) + kc * 256, d = SWZ ? db : 0;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(tile + x.tr[d % NTR][0] + add));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(tile + x.tr[d % NTR][1] + add));
    const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, both);
  }
};

// Sums over the contraction slice of a B operand of the 32 x 32 x 16 instruction, for all 32 columns, by ONE 16 x 16 x 32
// instruction: that one takes the lanes of columns n and n + 16 for the same column, and this A operand (ones where row and
// contraction group agree) keeps them apart, so that element 0 of the result is the sum of the lane's own column.
__device__ inline bf16x8 column_ones() {
  const int l = threadIdx.x & 63;
  const float w1 = __builtin_bit_cast(float, (l >> 2 & 1) == (l >> 4 & 1) ? 0x3F803F80u : 0u);
  f32x4 w = {w1, w1, w1, w1};
  asm volatile("" : "+v"(w));
  return __builtin_bit_cast(bf16x8, w);
}

// Maximum over the two lanes of a column, in both.
__device__ inline float t32_column_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float max16(const f32x16 &x) {
  float m = x[0];
#pragma unroll
  for (int i = 1; i < 16; ++i) m = fmaxf(m, x[i]);
  return m;
}

// Store an accumulator tile (columns x D, rows of a transposed operand as above) as bf16 rows: lane n and n + 32 hold column n's
// dims in 16-byte pieces (register half k of block db: dims 32*db + 16*k + 8*h .. +7).  Exchanging the pieces k = 0, 1 between
// lanes 16 apart leaves 64 contiguous bytes of 16 rows in an instruction, and where a row has two such groups trading them between
// lanes 8 apart 128 bytes of 8 rows: whole cache lines go out at once.  `row`: this lane's column.  Stored under no condition
// (columns that stand for nothing have a spare row), so that the compiler can count the stores and a wait for loads issued before
// them does not wait for them as well.  Nontemporal: the rows are read once, much later.
template <int D>
__device__ inline void t32_store_rows(bf16_t *base, uint32_t row, const f32x16 (&o)[D / 32]) {
  typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
  const int lane = threadIdx.x & 63, n16 = lane & 15, quad = lane >> 4;
  const int off = 8 * ((quad & 1) << 1 | quad >> 1);  // dims of quad's piece after the exchange
  const auto rr = __builtin_amdgcn_permlane16_swap(row, row, false, false);  // rows of columns 0 .. 15, of 16 .. 31
  u32x4 g[2][D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db) {
    bf16x8 x0, x1;
#pragma unroll
    for (int i = 0; i < 8; ++i) { x0[i] = (__bf16)o[db][i]; x1[i] = (__bf16)o[db][8 + i]; }
    const u32x4 w0 = __builtin_bit_cast(u32x4, x0), w1 = __builtin_bit_cast(u32x4, x1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const auto s = __builtin_amdgcn_permlane16_swap(w0[i], w1[i], false, false);
      g[0][db][i] = s[0];
      g[1][db][i] = s[1];
    }
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {  // columns 0 .. 15, 16 .. 31
    const unsigned r = rr[c];
    if constexpr (D % 64 == 0) {
      auto upper = [](unsigned keep, unsigned from) {  // lanes n16 >= 8 take `from` of the lane 8 below
        return (unsigned)__builtin_amdgcn_update_dpp((int)keep, (int)from, 0x128, 0xF, 0xC, false);
      };
      auto lower = [](unsigned keep, unsigned from) {  // lanes n16 < 8 take `from` of the lane 8 above
        return (unsigned)__builtin_amdgcn_update_dpp((int)keep, (int)from, 0x128, 0xF, 0x3, false);
      };
      const unsigned r0 = upper(r, r), r1 = lower(r, r);
      const int o2 = off + 32 * (n16 >> 3);
#pragma unroll
      for (int hh = 0; hh < D / 64; ++hh) {
        u32x4 x, y;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          x[i] = upper(g[c][2 * hh][i], g[c][2 * hh + 1][i]);
          y[i] = lower(g[c][2 * hh + 1][i], g[c][2 * hh][i]);
        }
        __builtin_nontemporal_store(x, reinterpret_cast<u32x4 *>(base + (size_t)r0 * D + 64 * hh + o2));
        __builtin_nontemporal_store(y, reinterpret_cast<u32x4 *>(base + (size_t)r1 * D + 64 * hh + o2));
      }
    } else {
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
        __builtin_nontemporal_store(g[c][db], reinterpret_cast<u32x4 *>(base + (size_t)r * D + 32 * db + off));
    }
  }
}

// Copy rows r0 .. r0 + n - 1 of two row-major arrays (already offset to the KV group; `stride` elements between rows) into LDS
// tiles, zeros behind them up to a whole tile: products with rows that are not the block's are exact zeros.
template <int D, bool SWZ, int NTHR>
__device__ inline void t32_stage2(const bf16_t *xa, const bf16_t *xb, uint32_t stride, int r0, int n, unsigned char *ta, unsigned char *tb) {
  using T = T32<D, SWZ>;
  const int total = (n + 31) / 32 * T::ITEMS;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // (or the offsets below stay in registers from one segment of a block to the next)
  for (int i0 = 0; i0 < total; i0 += 4 * NTHR) {
    bf16x8 ra[4], rb[4];
    int off[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int it = i0 + u * NTHR + tid;
      const int row = it / T::SEGS, seg = it % T::SEGS;
      // (loads under no condition, so that all of them are in flight together)
      const uint32_t src = (uint32_t)(r0 + min(row, n - 1)) * stride + (uint32_t)(seg * 8);
      ra[u] = ld8(xa + src);
      rb[u] = ld8(xb + src);
      if (row >= n) ra[u] = rb[u] = zero8();
      off[u] = it < total ? row / 32 * T::BYTES + T::off(row % 32, seg) : -1;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (off[u] >= 0) {
        *reinterpret_cast<bf16x8 *>(ta + off[u]) = ra[u];
        *reinterpret_cast<bf16x8 *>(tb + off[u]) = rb[u];
      }
  }
}
