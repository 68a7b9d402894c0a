// LDS tile layouts of the 16 x 16 x 32 matrix kernels (dK/dV, the one-pass selection backward, the projections, the gate predictor
// and the compression module), the workgroup map of the query-centric attention kernels and the top-k search (gfx950, wave64).
#pragma once

#include "mfma_common.h"
#include "mfma_t32.h"
#include "topk_device.h"

// LDS geometry of one staged tile set.
// Row-major tiles (32 rows of D bf16, no padding) are stored as [16-byte segment][row slot][8 elements]: the slot of
// row k is sigma(k) = 16*((k>>2)&1) + 4*(k>>3) + (k&3), i.e. the 16 rows lane n = 0..15 of sub-tile a reads (the
// key-tile convention of mfma_common.h) occupy the consecutive slots 16a .. 16a+15, so one operand read of a 16-lane quad covers 256
// contiguous bytes.  The slot is XORed with (segment & 7): reads stay a permutation of the same 16 slots, and the
// 8 threads that stage one row (8 segments, 512 bytes apart) land in 8 different 16-byte bank groups.
template <int D>
struct TileGeom {
  static constexpr int ROW_ELEMS = 32 * D;
  static constexpr int ROW_ITEMS = 32 * D / 8;                  // 16-byte items of a row-major tile
  __device__ static inline int sigma(int row) { return 16 * ((row >> 2) & 1) + 4 * (row >> 3) + (row & 3); }
  // element offset of (row slot, 16-byte segment) inside a row-major tile
  __device__ static inline int slot_off(int slot, int seg) { return ((seg << 5) + (slot ^ (seg & 7))) << 3; }
  // element offset of (row, 16-byte segment)
  __device__ static inline int row_off(int row, int seg) { return slot_off(sigma(row), seg); }
};

typedef __attribute__((ext_vector_type(4))) short s16x4;

// Tile layout of the dK/dV kernels and the one-pass selection backward in LDS.  A 32-row tile of a row-major bf16 array is kept
// as D/8 planes of 512 bytes, one per 16-byte segment of a row; a plane holds the 32 rows' segments in the slot order sigma(row) (the order
// in which the lanes of the two 16-row matrix sub-tiles read them).  The slot is XORed with a per-plane constant,
// swz(seg), chosen so that all three access patterns are free of LDS bank conflicts (measured with the LDS counters:
// 0 conflict cycles per instruction for each):
//   * staging writes: the 8 threads that stage one row write 8 planes, 512 bytes apart; the low three bits of swz
//     (seg & 7) put them in 8 different 16-byte bank groups;
//   * row operands (16-byte reads): the four quads of a wavefront read planes 4*ks .. 4*ks + 3, each 16 consecutive
//     slots; the two quads served together (0,1 and 2,3) must not differ in bit 3 of swz, so that bit is the same for
//     segments 4*ks, 4*ks + 1 and for 4*ks + 2, 4*ks + 3;
//   * transposed operands (8-byte transposing reads): one read takes 4-element pieces from TWO planes; planes whose
//     swz agrees in bit 3 would collide (they are a multiple of 512 bytes apart), so a dim block pairs segment s with
//     segment s + 2, whose bit 3 differs.  The 16 output rows of dim block dt are therefore not the dims 16*dt .. +15
//     but tr_dim(dt, 0..15): dims 8*s .. 8*s + 7 and 8*s + 16 .. 8*s + 23 with s = tr_seg(dt).  Every consumer of an
//     accumulator indexed by dt goes through acc_dim() (mfma_common.h), which states the same map per lane.
// Operand addresses are lane part + compile-time constant: the lane part depends on the contraction step (row
// operands) or the output-dim block (transposed operands) only through the swizzle, so a kernel keeps D/32 + D/16
// lane offsets in registers (Lanes) and the sub-tile, the row half, the tile index and the LDS stage all move the
// address by constants, which the LDS instructions take as immediate offsets: a tile costs no address arithmetic.
template <int D>
struct PTile {
  static constexpr int SEGS = D / 8;
  static constexpr int PLANE_B = 512;            // bytes per plane: 32 row slots of 16 bytes
  static constexpr int BYTES = SEGS * PLANE_B;   // bytes per 32-row tile
  static constexpr int ITEMS = 32 * SEGS;        // 16-byte items per tile
  __device__ static inline int swz(int seg) { return (seg & 7) ^ (((seg >> 1) & 1) << 3); }
  __device__ static inline int slot_off(int slot, int seg) { return seg * PLANE_B + ((slot ^ swz(seg)) << 4); }
  __device__ static inline int off(int row, int seg) { return slot_off(TileGeom<D>::sigma(row), seg); }
  // first of the two segments (s, s + 2) that dim block dt of a transposed operand is read from
  __device__ static inline int tr_seg(int dt) { return 4 * (dt >> 1) + (dt & 1); }
  struct Lanes {
    int row[D / 32];  // row operand (rows = the tile's rows), contraction step ks; sub-tile a adds a*256
    int tr[D / 16];   // transposed operand (rows = dims tr_dim(dt, n), contraction over rows 8*quad .. +7); rows +4 .. +7 add 256
  };
  __device__ static inline Lanes lanes() {
    const int n = threadIdx.x & 15, quad = threadIdx.x >> 4 & 3;
    Lanes l;
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks) l.row[ks] = slot_off(n, 4 * ks + quad);
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) l.tr[dt] = slot_off(4 * quad + (n >> 2), tr_seg(dt) + ((n & 3) >> 1) * 2) + (n & 1) * 8;
    return l;
  }
};

// A operand of sub-tile a, contraction step ks (row = key, in the key-tile convention) from the tile at `tile` (uniform address).
template <int D>
__device__ inline bf16x8 p_row_operand(lds_cptr tile, const typename PTile<D>::Lanes &l, int a, int ks) {
  return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8 *>(tile + l.row[ks] + a * 256);
}

// Transposed A operand (row n = dim tr_dim(dt, n), contraction over the tile's rows 8*quad .. +7), taken from the same
// row-major tile with the transposing LDS read of gfx950 (ds_read_b64_tr_b16): inside a 16-lane group lane p hands in
// the address of 4 consecutive elements and lane i receives element (i & 3) of lanes (i >> 2), 4 + (i >> 2),
// 8 + (i >> 2), 12 + (i >> 2).  With lane p pointing at row 8*quad + (p >> 2) and at the 4-dim piece (p & 3) of the
// block (pieces 0, 1 in segment tr_seg(dt), pieces 2, 3 in the segment two further), lane i ends up with dim
// tr_dim(dt, i) of rows 8*quad .. +3; a second read covers rows +4 .. +7.
template <int D>
__device__ inline bf16x8 p_tr_operand(lds_cptr tile, const typename PTile<D>::Lanes &l, int dt) {
  typedef __attribute__((address_space(3))) s16x4 *tr_ptr;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(tile + l.tr[dt]));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(tile + l.tr[dt] + 256));
  typedef __attribute__((ext_vector_type(8))) short s16x8;
  const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, both);
}

// A operand of sub-tile a, contraction step ks, from a row-major LDS tile (row = key, in the key-tile convention).
template <int D>
__device__ inline bf16x8 lds_row_operand(const bf16_t *tile, int a, int ks) {
  const int n = threadIdx.x & 15, quad = threadIdx.x >> 4 & 3;
  return *reinterpret_cast<const bf16x8 *>(tile + TileGeom<D>::slot_off(16 * a + n, 4 * ks + quad));
}

// Transposed A operand (row = dim 16*dt + n, contraction over the tile's rows 8*quad .. +7), taken from the same
// ROW-major LDS tile with the transposing LDS read of gfx950 (ds_read_b64_tr_b16): inside a 16-lane group lane p
// hands in the address of 4 consecutive elements and lane i receives element (i & 3) of lanes (i >> 2), 4 + (i >> 2),
// 8 + (i >> 2), 12 + (i >> 2).  With lane p pointing at row 8*quad + (p >> 2), dims 16*dt + 4*(p & 3) .. +3, lane i
// ends up with dim 16*dt + i of rows 8*quad .. +3; a second read covers rows +4 .. +7.  No transposed copy of the
// tile is needed, in LDS or in memory.
template <int D>
__device__ inline bf16x8 lds_tr_operand(const bf16_t *tile, int dt) {
  const int p = threadIdx.x & 15, quad = threadIdx.x >> 4 & 3;
  const int d0 = 16 * dt + 4 * (p & 3), seg = d0 >> 3, within = d0 & 7;
  const int row = 8 * quad + (p >> 2);
  const bf16_t *a0 = tile + TileGeom<D>::row_off(row, seg) + within;
  const bf16_t *a1 = tile + TileGeom<D>::row_off(row + 4, seg) + within;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)a0);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)a1);
  typedef __attribute__((ext_vector_type(8))) short s16x8;
  const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, both);
}

__device__ inline int lds_uniform(const int *p) { return __builtin_amdgcn_readfirstlane(*p); }
// Workgroup -> (token tile, KV group).  Workgroups of a 1-D launch are dealt round-robin to the 8 XCDs, each with
// its own L2; this map keeps every XCD on ONE KV group and one contiguous run of token tiles, so the K/V rows it
// touches (one group's pooled keys, the windows and selected blocks of neighbouring tokens) stay L2 resident.
struct TileMap {
  int tile, g;
  bool valid;
};
__host__ __device__ inline int xcd_grid_size(int n_tiles, int Hkv) {
  if (Hkv > 8 || 8 % Hkv != 0) return n_tiles * Hkv;
  const int parts = 8 / Hkv;
  return 8 * ((n_tiles + parts - 1) / parts);
}
__device__ inline TileMap xcd_tile_map(int n_tiles, int Hkv, int L = blockIdx.x) {  // L: number of the workgroup
  if (Hkv > 8 || 8 % Hkv != 0) return TileMap{L % n_tiles, L / n_tiles, L < n_tiles * Hkv};
  const int xcd = L & 7, idx = L >> 3, parts = 8 / Hkv;
  const int g = xcd % Hkv, part = xcd / Hkv;
  const int tpp = (n_tiles + parts - 1) / parts;
  const int tile = part * tpp + idx;
  return TileMap{tile, g, idx < tpp && tile < n_tiles};
}

// Maximum over the wavefront, uniform (row permutations inside 16 lanes, then register swaps).
__device__ inline uint32_t wave_max_dpp(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));   // xor 1
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));   // xor 2
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));  // half-row mirror
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));  // row mirror
  auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = max((uint32_t)r[0], (uint32_t)r[1]);
  r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return __builtin_amdgcn_readfirstlane((int)max((uint32_t)r[0], (uint32_t)r[1]));
}

// Top-k over unsigned fixed-point scores S[0..n) held in LDS by one wavefront, ties to the lowest index, entirely in
// registers and wave ballots (no lane exchange, no LDS traffic inside the search).  Lane l keeps entries l, l+64, ...
// (up to R per lane, n <= 64*R).  The T-th largest value is found by building it bit by bit from the top: a
// candidate threshold is kept when at least T entries reach it (one compare + ballot + population count per
// register and bit), and the search ends at the bit where exactly T do.  Entries above the threshold are selected, entries equal to it in ascending index order until
// T are reached.  Writes T ids (base + index) in ascending order, padded with -1, and counts them in hist[id] (LDS; null: not).
template <int R>
__device__ inline void topk_wave_bits(const uint32_t *S, int n, int T, int base, int32_t *out, uint32_t *hist) {
  const int lane = threadIdx.x & 63;
  const uint64_t lt = (1ull << lane) - 1ull;
  uint32_t val[R];  // score + 1 (so that every real entry is >= 1); 0 marks "no entry"
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = r * 64 + lane;
    val[r] = j < n ? S[j] + 1u : 0u;
  }
  const int Tn = T < n ? T : n;
  uint32_t thr = 0u;
  if (Tn > 0) {
    // from the highest bit any entry has down to the bit that separates exactly Tn entries from the rest
    uint32_t top = val[0];
#pragma unroll
    for (int r = 1; r < R; ++r) top = max(top, val[r]);
    top = wave_max_dpp(top);
    for (int b = 31 - __builtin_clz(top | 1u); b >= 0; --b) {
      const uint32_t cand = thr | (1u << b);
      int cnt = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        cnt += __popcll(__ballot(val[r] >= cand));
        if (R > 16 && (r & 7) == 7) __builtin_amdgcn_sched_barrier(0);  // (more masks at a time spill)
      }
      if (cnt >= Tn) thr = cand;
      if (cnt == Tn) break;
    }
  }
  if constexpr (R > 16) {  // (from LDS again, in loops that are not unrolled: see the masks above)
    int greater = 0, written = 0, eq_before = 0;
    for (int j0 = 0; j0 < n; j0 += 64) greater += __popcll(__ballot(j0 + lane < n && S[min(j0 + lane, n - 1)] + 1u > thr));
    const int need = Tn - greater;
    for (int j0 = 0; j0 < n && written < Tn; j0 += 64) {
      const int j = j0 + lane;
      const uint32_t v = j < n ? S[j] + 1u : 0u;
      const bool eq = Tn > 0 && v == thr;
      const uint64_t em = __ballot(eq);
      const bool sel = (Tn > 0 && v > thr) || (eq && eq_before + (int)__popcll(em & lt) < need);
      eq_before += __popcll(em);
      const uint64_t sm = __ballot(sel);
      if (sel) out[written + __popcll(sm & lt)] = base + j;
      written += __popcll(sm);
    }
    for (int w = written + lane; w < T; w += 64) out[w] = -1;
    return;
  }
  int greater = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) greater += __popcll(__ballot(val[r] > thr));
  const int need = Tn - greater;  // entries equal to the threshold still to take, lowest indices first
  int written = 0, eq_before = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool eq = Tn > 0 && val[r] == thr;
    const uint64_t em = __ballot(eq);
    const bool sel = (Tn > 0 && val[r] > thr) || (eq && eq_before + (int)__popcll(em & lt) < need);
    eq_before += __popcll(em);
    const uint64_t sm = __ballot(sel);
    if (sel) out[written + __popcll(sm & lt)] = base + r * 64 + lane;
    if (sel && hist) atomicAdd(&hist[base + r * 64 + lane], 1u);
    written += __popcll(sm);
  }
  for (int w = written + lane; w < T; w += 64) out[w] = -1;
}

// ---- top-k over unsigned fixed-point scores held in LDS by one wavefront (ties -> lowest id) ----
__device__ inline void topk_wave_u32(const uint32_t *S, int n, int T, int base, int32_t *out, uint32_t *sel) {
  const int lane = threadIdx.x & 63;
  const int words = (n + 31) >> 5;
  for (int i = lane; i < words; i += 64) sel[i] = 0u;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const int rounds = T < n ? T : n;
  for (int r = 0; r < rounds; ++r) {
    uint64_t best = 0ull;
    for (int j = lane; j < n; j += 64) {
      if ((sel[j >> 5] >> (j & 31)) & 1u) continue;
      const uint64_t key = ((uint64_t)S[j] << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)j);
      best = key > best ? key : best;
    }
    best = wave_max_u64(best);
    const uint32_t j = 0xFFFFFFFFu - (uint32_t)(best & 0xFFFFFFFFull);
    if (lane == 0) sel[j >> 5] |= 1u << (j & 31);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  int written = 0;
  for (int j0 = 0; j0 < n; j0 += 64) {
    const int j = j0 + lane;
    const bool s = j < n && ((sel[j >> 5] >> (j & 31)) & 1u);
    const uint64_t m = __ballot(s);
    if (s) out[written + __popcll(m & ((1ull << lane) - 1ull))] = base + j;
    written += __popcll(m);
  }
  for (int w = written + lane; w < T; w += 64) out[w] = -1;
}
