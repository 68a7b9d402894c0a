// 32 x 32 x 16 matrix tiles of the attention kernels (gfx950, wave64, v_mfma_f32_32x32x16_bf16): LDS tile layout, operands,
// softmax sums and row stores.
//
// Operand convention of the instruction (h = lane >> 5, n = lane & 31):
//   A (32 x 16): the lane supplies row n, contraction indices 8*h .. +7;  B (16 x 32): column n, the same indices
//   C/D (32 x 32 fp32): the lane holds column n, rows 8*(i >> 2) + 4*h + (i & 3), i = 0 .. 15
// A wavefront keeps 32 query columns and walks over tiles of 32 keys.  Scores are formed transposed (keys x queries) from key rows
// in the order t32_order (bits 2 and 3 of row and key change places), so that registers 8*kc .. +7 of a lane are, for its query, the
// consecutive keys 16*kc + 8*h .. +7: the contraction slice kc (16 keys) of the next product, as the B operand wants it.
//
// Why 32 columns and not 16: an operand taken from LDS (1 KB) feeds a matrix instruction of 32 cycles instead of 16.  With 16
// columns the four SIMDs of a compute unit ask for as many LDS cycles as they spend matrix cycles, and the kernels wait for LDS
// whatever their vector work is.
#pragma once

#include "mfma_common.h"

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef const __attribute__((address_space(3))) unsigned char *lds_cptr;

__device__ inline f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
__device__ inline f32x16 splat16(float x) {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = x;
  return z;
}
// Key of row r of a tile, and row of key r; key of register i of a score tile.
__device__ inline int t32_order(int r) { return (r & 0x13) | (r >> 1 & 4) | (r << 1 & 8); }
__device__ inline int t32_key(int i) { return 16 * (i >> 3) + 8 * (threadIdx.x >> 5 & 1) + (i & 7); }
// Row of register i of any other accumulator tile.
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
    int row[NROW];    // row operand (rows in the order of t32_order), contraction step ks (ks & 1 without SWZ)
    int tr[NTR][2];   // transposed operand: keys +0 .. 3 and +4 .. 7 of the lane's eight, dim block db (the first without SWZ)
  };
  // The 32 rows of a transposed operand are the dims of block db in the order that leaves a lane with 8 consecutive dims in
  // registers 0 .. 7 (32*db + 8*h ..) and in 8 .. 15 (32*db + 16 + 8*h ..): bits 2 and 3 of row and dim change places.
  __device__ static inline Lanes lanes() {
    const int l = threadIdx.x & 63, h = l >> 5, p = l & 3, r = (l & 15) >> 2;
    Lanes x;
#pragma unroll
    for (int ks = 0; ks < NROW; ++ks) x.row[ks] = off(t32_order(l & 31), 2 * ks + h);
#pragma unroll
    for (int db = 0; db < NTR; ++db)
#pragma unroll
      for (int k = 0; k < 2; ++k) x.tr[db][k] = off(8 * h + 4 * k + r, 4 * db + 2 * (l >> 4 & 1) + (p & 1)) + 8 * (p >> 1);
    return x;
  }
  // A or B operand: rows of the tile in the order of t32_order, dims 16*ks + 8*h .. +7
  __device__ static inline bf16x8 row(lds_cptr tile, const Lanes &x, int ks) {
    const int o = SWZ ? x.row[ks % NROW] : x.row[ks & 1] + (ks >> 1) * 2048;
    return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8 *>(tile + o);
  }
  // A operand: dims of block db, contraction over the keys of slice kc (ds_read_b64_tr_b16: of a group of 16 lanes lane 4*r + p
  // hands in the address of 4 dims of row r, and lane i receives dim i of the four rows)
  __device__ static inline bf16x8 tr(lds_cptr tile, const Lanes &x, int db, int kc) {
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

// Transposed scores of 32 query columns over a 32-key LDS tile: element i = key t32_key(i), column n.  s: what they start from.
template <int D, bool SWZ>
__device__ inline f32x16 t32_scores(const bf16x8 (&qop)[D / 16], lds_cptr kt, const typename T32<D, SWZ>::Lanes &ln, f32x16 s) {
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) s = mfma32(T32<D, SWZ>::row(kt, ln, ks), qop[ks], s);
  return s;
}

// Scores of the tile whose first key is kb, minus infinity for the keys outside [lo, hi).  (Replaced, not added to: a tile at the end
// of a range holds keys of the next one, whose product with any query may have left the range of the floats.)
__device__ inline void t32_only_keys(f32x16 &s, int kb, int lo, int hi) {
  const int rel = kb - lo;
  const unsigned len = (unsigned)(hi - lo);
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if ((unsigned)(rel + t32_key(i)) >= len) s[i] = -INFINITY;  // lo <= key < hi as one comparison
}

// The sum of a B operand's eight entries by products with two bf16 ones (32-bit sums), onto c.
__device__ inline float bf16_ones() { return in_vgpr(__builtin_bit_cast(float, 0x3F803F80u)); }
__device__ inline float sum8(bf16x8 p, float ones, float c) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    c = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{p[2 * j], p[2 * j + 1]}, __builtin_bit_cast(bf16x2, ones), c, false);
  return c;
}
// Sum over the two lanes of a column, in both.
__device__ inline float t32_column_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sums of the probabilities of 32 columns, in the same bf16 rounding the numerator uses.  In parts: two per lane, four per column.
struct SumParts {
  float part[2], ones;
  __device__ inline SumParts() { ones = bf16_ones(); }
  __device__ inline void clear() { part[0] = part[1] = 0.f; }
  __device__ inline void add(bf16x8 p, int kc, bool first) { part[kc] = sum8(p, ones, first ? 0.f : part[kc]); }
  __device__ inline void scale(float a) { part[0] *= a; part[1] *= a; }
  __device__ inline float mine() const { return part[0] + part[1]; }
  __device__ inline float total() const { return t32_column_sum(mine()); }
};
// On the matrix pipe, bit for bit what one 16 x 16 x 32 product with ones gives over the tile's keys in order: two
// register swaps bring the slices of 16 columns together, so that a product of that shape sums the tile's 32 keys.  For the
// compression branch: its normaliser scales the selection scores, and a top-k among near-equal scores depends on their last bits.
// (A 32 x 32 x 16 product with ones gives the same but takes 16 registers, which the walk has not got: 1400 us for 1370 at 62k
// tokens; sums in parts as above 1290 us, with the lse of most rows off in the last bit and some five rows of 100000 choosing
// another of two blocks.)
struct SumInOrder {
  f32x4 sum[2];  // element 0: columns 0 .. 15, columns 16 .. 31
  bf16x8 ones, before;
  __device__ inline SumInOrder() {
    const float w1 = __builtin_bit_cast(float, 0x3F803F80u);
    f32x4 w = {w1, w1, w1, w1};
    asm volatile("" : "+v"(w));  // (opaque, or it is rebuilt with four moves in front of every use)
    ones = __builtin_bit_cast(bf16x8, w);
  }
  __device__ inline void clear() { sum[0] = sum[1] = f32x4{0.f, 0.f, 0.f, 0.f}; }
  __device__ inline void add(bf16x8 p, int kc, bool first) {
    if (kc == 0) {
      before = p;
      return;
    }
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
    const u32x4 x = __builtin_bit_cast(u32x4, before), y = __builtin_bit_cast(u32x4, p);
    u32x4 lo, hi;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const auto h = __builtin_amdgcn_permlane32_swap(x[i], y[i], false, false);
      const auto q = __builtin_amdgcn_permlane16_swap(h[0], h[1], false, false);
      lo[i] = q[0];
      hi[i] = q[1];
    }
    if (first) clear();
    sum[0] = mfma16(ones, __builtin_bit_cast(bf16x8, lo), sum[0]);
    sum[1] = mfma16(ones, __builtin_bit_cast(bf16x8, hi), sum[1]);
  }
  __device__ inline void scale(float a) {
    // (the factors of the other 16 columns are in the lanes 16 away)
    const auto f = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(a), false, false);
    sum[0][0] *= __uint_as_float(f[0]);
    sum[1][0] *= __uint_as_float(f[1]);
  }
  __device__ inline float mine() const { return threadIdx.x & 16 ? sum[1][0] : sum[0][0]; }
  __device__ inline float total() const { return mine(); }
};

// Softmax state of 32 query columns (Algorithm 1's o, l, m): unnormalised output (transposed), sum, reference exponent in log2 units.
template <int D, class Sum>
struct T32State {
  f32x16 o[D / 32];
  Sum l;
  float m;
};
template <int D, class Sum>
__device__ inline void t32_clear(T32State<D, Sum> &st) {
#pragma unroll
  for (int db = 0; db < D / 32; ++db) st.o[db] = splat16(0.f);
  st.l.clear();
  st.m = -INFINITY;
}

// One step of the softmax (Algorithm 1, inner loop body) over a tile with raw scores s.  The reference exponent of a column is the
// maximum of its first tile (FIRST) and stays: later tiles cost a fused multiply-add, an exponential and half a conversion
// per score, no maximum and no rescaling.  The result does not depend on the reference as long as nothing leaves the range of the
// floats, which the caller checks on the finished sums (t32_in_range).
template <int D, bool SWZ, bool FIRST, class Sum>
__device__ inline void t32_softmax(T32State<D, Sum> &st, const f32x16 &s, lds_cptr vt, const typename T32<D, SWZ>::Lanes &ln, float sl2) {
  if (FIRST) st.m = t32_column_max(max16(s)) * sl2;
#pragma unroll
  for (int kc = 0; kc < 2; ++kc) {
    const bool fresh = FIRST && kc == 0;  // (no registers to clear: the products start from a constant)
    bf16x8 p;
#pragma unroll
    for (int j = 0; j < 8; ++j) p[j] = (__bf16)fast_exp2(__builtin_fmaf(s[8 * kc + j], sl2, -st.m));
    st.l.add(p, kc, FIRST);
#pragma unroll
    for (int db = 0; db < D / 32; ++db) st.o[db] = mfma32(T32<D, SWZ>::tr(vt, ln, db, kc), p, fresh ? splat16(0.f) : st.o[db]);
  }
}

// The first tile's maximum contributes 1 to the sum, so nothing that counts is lost below; a sum under 2^60 leaves room for
// values of the same size.  A sum that is no number (a first tile all of whose scores are minus infinity, a score of plus infinity) is
// out of range as well: the comparison is one of the bits, as integers, because these files are compiled as if NaN did not occur and
// the comparison of floats would come out either way.
template <int D, class Sum>
__device__ inline bool t32_in_range(const T32State<D, Sum> &st) {
  uint32_t bits = __float_as_uint(st.l.mine());
  asm volatile("" : "+v"(bits));
  return bits < 0x5D800000u;  // 2^60; sums are not negative
}

// The same step with a running maximum (-inf for keys that do not count): the reference is raised when some
// score exceeds it by more than 8 log2 units, so that every exponent stays below 8.
template <int D, bool SWZ, class Sum>
__device__ inline void t32_softmax_running(T32State<D, Sum> &st, const f32x16 &s, lds_cptr vt, const typename T32<D, SWZ>::Lanes &ln, float sl2) {
  const float pm = max16(s) * sl2;
  if (__any(pm > st.m + 8.f)) {
    const float mn = fmaxf(st.m, t32_column_max(pm));
    const float alpha = mn == -INFINITY ? 1.0f : fast_exp2(st.m - mn);
    st.l.scale(alpha);
    st.m = mn;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) st.o[db][i] *= alpha;
  }
  const float neg = st.m != -INFINITY ? -st.m : -INFINITY;
#pragma unroll
  for (int kc = 0; kc < 2; ++kc) {
    bf16x8 p;
#pragma unroll
    for (int j = 0; j < 8; ++j) p[j] = (__bf16)fast_exp2(__builtin_fmaf(s[8 * kc + j], sl2, neg));
    st.l.add(p, kc, false);
#pragma unroll
    for (int db = 0; db < D / 32; ++db) st.o[db] = mfma32(T32<D, SWZ>::tr(vt, ln, db, kc), p, st.o[db]);
  }
}

// What the score accumulators of a range's last tile start from: 0, and -inf for the keys that do not count (32 floats of LDS).
__device__ inline f32x16 t32_tail(const float *tail) {
  f32x16 s;
  int first = t32_key(0);
  asm volatile("" : "+v"(first));  // (or the 16 values stay in registers between the steps)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f32x4 x = *reinterpret_cast<const f32x4 *>(tail + first + 16 * (i >> 1) + 4 * (i & 1));
#pragma unroll
    for (int j = 0; j < 4; ++j) s[4 * i + j] = x[j];
  }
  return s;
}
__device__ inline void t32_write_tail(float *tail, int left) {
  if (threadIdx.x < 32) tail[threadIdx.x] = (int)threadIdx.x < left ? 0.f : -INFINITY;
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

// Global sources of a tile set: row-major arrays, already offset to the KV group; `stride` elements between rows (whole arrays stay
// below 2^31 elements).
template <int NROW>
struct T32Src {
  const bf16_t *row[NROW];
  uint32_t stride;
};

// Walk of a workgroup over the rows [rs, re) of NROW arrays in steps of STEP rows: 32-row tiles (one of each array; the arrays may
// be consecutive tiles of one, with STEP a multiple of 32) go global -> registers -> LDS once per workgroup, loads one step ahead (a
// second register set costs more than it hides: spills), two LDS stages and one barrier per step.  tile(first tile of the stage, first
// row) consumes a stage.  Rows past re are read as they lie in memory (padded arrays) and are the consumer's to mask.
// PAIRS: the loop takes two steps at a time and the last of an odd number stands behind it, instead of a way out between the two: the accumulators
// of a softmax then stay in their registers (32 register moves per two tiles otherwise, and more spilled).  The dQ kernel keeps them either way,
// and has no register for the third copy of its tile.
template <int D, int NROW, int NTHR, int STEP, bool PAIRS = true, class Tile>
__device__ inline void t32_pipeline(const T32Src<NROW> &src, unsigned char *stage0, int rs, int re, Tile tile) {
  using T = T32<D, true>;
  constexpr int NI = (T::ITEMS + NTHR - 1) / NTHR;
  static_assert(T::ITEMS % NTHR == 0 || NI == 1, "whole tiles at a time");
  const bool mine = T::ITEMS >= NTHR || (int)threadIdx.x < T::ITEMS;
  const int row0 = threadIdx.x / T::SEGS, seg = threadIdx.x % T::SEGS;
  bf16x8 r[NROW][NI];
  auto load = [&](int kb) {
    if (!mine) return;
#pragma unroll
    for (int a = 0; a < NROW; ++a)
#pragma unroll
      for (int i = 0; i < NI; ++i)
        r[a][i] = ld8(src.row[a] + ((uint32_t)(kb + row0 + i * (NTHR / T::SEGS)) * src.stride + (uint32_t)(seg * 8)));
  };
  auto step = [&](int buf, int kb) {
    unsigned char *st = stage0 + buf * NROW * T::BYTES;
    if (mine)
#pragma unroll
      for (int a = 0; a < NROW; ++a)
#pragma unroll
        for (int i = 0; i < NI; ++i) *reinterpret_cast<bf16x8 *>(st + a * T::BYTES + T::off(row0 + i * (NTHR / T::SEGS), seg)) = r[a][i];
    if (kb + STEP < re) load(kb + STEP);
    __syncthreads();
    tile((lds_cptr)st, kb);
  };
  if (rs < re) load(rs);
  int kb = rs;
  for (; PAIRS ? kb + STEP < re : kb < re; kb += 2 * STEP) {
    step(0, kb);
    if (!PAIRS && kb + STEP >= re) break;
    step(1, kb + STEP);
  }
  if (PAIRS && kb < re) step(0, kb);
  __syncthreads();
}

// Workgroup of NW wavefronts: 32*NW query rows = consecutive sorted tokens x the heads of one KV group, 32 per wavefront.
struct QCol {
  int slot, pos, tok, h;  // token slot inside the workgroup, sorted position, caller index, head
  bool valid;             // columns past the last token repeat it and are not stored
};
// (Looked up again where it is needed after a walk, through an opaque thread number: held across the walk it takes registers that
// the walk has not got.)
__device__ inline QCol query_col(const MfmaView &v, int wg_pos0, int g) {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  const int row = (t >> 6) * 32 + (t & 31);
  QCol q;
  q.slot = row / v.hs;
  q.valid = wg_pos0 + q.slot < v.N;
  q.pos = min(wg_pos0 + q.slot, v.N - 1);
  q.tok = v.perm[q.pos];
  q.h = g * v.hs + row % v.hs;
  return q;
}
// The B operands of this lane's column from a caller-ordered array [N][Hq][D].
template <int D>
__device__ inline void load_col(const bf16_t *X, const MfmaView &v, const QCol &q, bf16x8 (&op)[D / 16]) {
  const bf16_t *src = X + ((size_t)q.tok * v.Hq + q.h) * D + 8 * (threadIdx.x >> 5 & 1);
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) op[ks] = ld8(src + 16 * ks);
}
