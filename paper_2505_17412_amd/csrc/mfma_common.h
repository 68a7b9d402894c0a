// Shared pieces of the bf16 MFMA kernels (gfx950, wave64, v_mfma_f32_16x16x32_bf16).
//
// Operand convention used throughout (hardware layout of the 16x16x32 instruction):
//   A (16 x 32): lane l supplies row (l & 15), contraction indices 8*(l >> 4) .. +7   (8 bf16 = 16 bytes)
//   B (32 x 16): lane l supplies column (l & 15), contraction indices 8*(l >> 4) .. +7
//   C/D (16 x 16 fp32): lane l holds column (l & 15), rows 4*(l >> 4) .. +3
// "quad" below is l >> 4, "n" is l & 15.
//
// Key-tile convention: a tile covers 32 consecutive rows kb..kb+31 of a key array, kb a multiple of 8.  It is
// processed as two 16-row sub-tiles whose row r maps to key kb + 8*(r >> 2) + 4*a + (r & 3) (a = sub-tile), so
// that after the two MFMAs lane l holds the eight CONSECUTIVE keys kb + 8*quad .. +7 of column n -- exactly
// the contraction slice the next MFMA wants from it as a B operand, with no cross-lane movement.
#pragma once

#include "ssa_internal.h"

typedef uint16_t bf16_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

__device__ inline bf16x8 ld8(const bf16_t *p) { return *reinterpret_cast<const bf16x8 *>(p); }
__device__ inline bf16x8 zero8() {
  bf16x8 z;
#pragma unroll
  for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.0f;
  return z;
}
__device__ inline f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// All-ones A operand of the matrix instruction (sums the 32 contraction entries of every column).  Build it once per
// kernel: the empty asm makes the value opaque, so it stays in its four registers instead of being rebuilt with
// three moves in front of every use.
__device__ inline bf16x8 ones_operand() {
  const float w1 = __builtin_bit_cast(float, 0x3F803F80u);  // two bf16 ones
  f32x4 w = {w1, w1, w1, w1};
  asm volatile("" : "+v"(w));
  return __builtin_bit_cast(bf16x8, w);
}
// A uniform factor of the per-score arithmetic, kept in a vector register: a vector instruction of three vector operands
// issues every 2.7 cycles with four wavefronts per SIMD, one with a scalar operand every 4.5 (measured on v_fma, v_fmac and
// v_mul alike).  The empty asm makes the value opaque, so it is not moved back to a scalar register.
__device__ inline float in_vgpr(float x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Waits for every load and store in flight (vmcnt(0), the other counters untouched).  The compiler knows the instruction: in front
// of a loop it lets the waits inside count on what an iteration leaves in flight, stores behind its loads among them.
__device__ inline void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// A value that is the same in all lanes, in a scalar register: branches and loops on it are scalar ones.
__device__ inline int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ inline int wave_min_i(int v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = min(v, __shfl_xor(v, off));
  return v;
}
__device__ inline int wave_max_i(int v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = max(v, __shfl_xor(v, off));
  return v;
}

// Sum over aligned groups of hs lanes (hs a power of two <= 16) inside each 16-lane row, with DPP lane
// permutations only (no LDS traffic): xor 1, xor 2 by quad permutes; once the lanes of a quad agree, the
// half-row and row mirrors act as xor 4 and xor 8.
template <int CTRL>
__device__ inline float dpp_add(float v) {
  return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
__device__ inline float group_sum(float v, int hs) {
  if (hs >= 2) v = dpp_add<0xB1>(v);    // quad_perm [1,0,3,2]
  if (hs >= 4) v = dpp_add<0x4E>(v);    // quad_perm [2,3,0,1]
  if (hs >= 8) v = dpp_add<0x141>(v);   // row_half_mirror
  if (hs >= 16) v = dpp_add<0x140>(v);  // row_mirror
  return v;
}

// Maximum over the four lanes 16 apart that share a column of a 16 x 16 tile, in all of them (two register swaps, no LDS).
__device__ inline float column_max(float v) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Dims of an accumulator whose rows came from a transposed tile operand.  The transposing LDS read takes the 16 rows
// of dim block dt from two 16-byte segments of a row that lie 32 bytes apart (see PTile in mfma_qc.h: that pairing is
// what keeps the read free of bank conflicts), so the block covers dims b .. b + 7 and b + 16 .. b + 23 with
// b = 32*(dt >> 1) + 8*(dt & 1).  tr_dim: dim of row n of the block; acc_dim: the first of the 4 consecutive dims that a
// lane of row group `quad` holds in its accumulator register of block dt (C layout: rows 4*quad .. +3).
__device__ inline int tr_dim(int dt, int n) { return 32 * (dt >> 1) + 8 * (dt & 1) + 16 * (n >> 3) + (n & 7); }
__device__ inline int acc_dim(int dt, int quad) { return tr_dim(dt, 4 * quad); }

// Store the accumulator tile of 16 query columns to row-major rows of D bf16 (base + row*D): on entry lane (n, quad) holds,
// for every dim block dt, the 4 dims acc_dim(dt, quad) .. +3 of column n, i.e. 8 bytes in each of D/16 places of its row.
// Within a pair of dim blocks (32 dims, dt = 2*h + dt0) the dim index is 16*quad1 + 8*dt0 + 4*quad0 + i (quad1, quad0 the
// bits of quad): exchanging dt0 with quad0 (one round of v_permlane16_swap: lanes 16 apart hold the same column) leaves
// every lane with 8 consecutive dims of its column, and the four lanes of a column with 32 dims.  Where a row has two such
// groups of 32 (D a multiple of 64), lanes n and n + 8 then trade one group against the other (a rotation by 8 inside the
// 16 lanes), so that each store instruction writes 128 contiguous bytes of 8 rows instead of 64 of 16: with several heads
// per KV head those rows are neighbours and whole cache lines go out at once.  `row`: this lane's row (column n); lanes
// with !valid take part in the exchanges and store nothing (the lanes of a column agree on valid).
template <int D>
__device__ inline void store_partial_row(bf16_t *base, uint32_t row, const f32x4 (&o)[D / 16], bool valid) {
  typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
  typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
  const int n = threadIdx.x & 15, quad = threadIdx.x >> 4 & 3;
  u32x4 g[D / 32];  // dims 32*h + 8*quad .. +7
#pragma unroll
  for (int h = 0; h < D / 32; ++h) {
    u32x2 w[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      bf16x4 x;
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = (__bf16)o[2 * h + j][i];
      w[j] = __builtin_bit_cast(u32x2, x);
    }
    // odd 16-lane rows of the first <-> even 16-lane rows of the second
    const auto a = __builtin_amdgcn_permlane16_swap(w[0][0], w[1][0], false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(w[0][1], w[1][1], false, false);
    g[h] = u32x4{a[0], b[0], a[1], b[1]};
  }
  // written once, read once much later by the merge kernel: streaming stores, so the rows do not push the query rows (which
  // every selected block reads again) out of the caches
  if constexpr (D % 64 == 0) {
    auto upper = [](unsigned keep, unsigned from) {  // lanes n >= 8 take `from` of lane n - 8
      return (unsigned)__builtin_amdgcn_update_dpp((int)keep, (int)from, 0x128, 0xF, 0xC, false);
    };
    auto lower = [](unsigned keep, unsigned from) {  // lanes n < 8 take `from` of lane n + 8
      return (unsigned)__builtin_amdgcn_update_dpp((int)keep, (int)from, 0x128, 0xF, 0x3, false);
    };
    const unsigned rv = valid ? row : ~0u;
    const unsigned r0 = upper(rv, rv), r1 = lower(rv, rv);  // rows of the first eight columns, of the last eight
    const int off = 8 * quad + 32 * (n >> 3);
#pragma unroll
    for (int h = 0; h < D / 64; ++h) {
      u32x4 x, y;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        x[i] = upper(g[2 * h][i], g[2 * h + 1][i]);
        y[i] = lower(g[2 * h + 1][i], g[2 * h][i]);
      }
      if (r0 != ~0u) __builtin_nontemporal_store(x, reinterpret_cast<u32x4 *>(base + (size_t)r0 * D + 64 * h + off));
      if (r1 != ~0u) __builtin_nontemporal_store(y, reinterpret_cast<u32x4 *>(base + (size_t)r1 * D + 64 * h + off));
    }
  } else {
#pragma unroll
    for (int h = 0; h < D / 32; ++h)
      if (valid) __builtin_nontemporal_store(g[h], reinterpret_cast<u32x4 *>(base + (size_t)row * D + 32 * h + 8 * quad));
  }
}

// Row of the A operand a lane feeds for sub-tile `a` of the key tile starting at kb.
__device__ inline int tile_key_row(int kb, int a) {
  const int r = threadIdx.x & 15;
  return kb + 8 * (r >> 2) + 4 * a + (r & 3);
}

// Device arrays of the block structure and the sorted K,V copies the kernels read.
struct MfmaView {
  const int32_t *perm, *tok_item, *tok_win, *cmp_start, *slc_start, *win_start, *cmp_slc, *cmp_batch, *slc_batch,
      *item_start;
  int N, Nc, Ns, Hq, Hkv, hs, T, s_max;
  float scale, sl2;  // softmax scale, scale * log2(e)
  // sorted copies (bf16), row-major [rows][Hkv][D]: token K, V and pooled K, V
  const bf16_t *Ks, *Vs, *Kc, *Vc;
};
