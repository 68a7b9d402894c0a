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

// Dims of an accumulator whose rows came from a transposed tile operand.  The transposing LDS read takes the 16 rows
// of dim block dt from two 16-byte segments of a row that lie 32 bytes apart (see PTile in mfma_qc.h: that pairing is
// what keeps the read free of bank conflicts), so the block covers dims b .. b + 7 and b + 16 .. b + 23 with
// b = 32*(dt >> 1) + 8*(dt & 1).  tr_dim: dim of row n of the block; acc_dim: the first of the 4 consecutive dims that a
// lane of row group `quad` holds in its accumulator register of block dt (C layout: rows 4*quad .. +3).
__device__ inline int tr_dim(int dt, int n) { return 32 * (dt >> 1) + 8 * (dt & 1) + 16 * (n >> 3) + (n & 7); }
__device__ inline int acc_dim(int dt, int quad) { return tr_dim(dt, 4 * quad); }

// Device arrays of the block structure and the sorted K,V copies the kernels read.
struct MfmaView {
  const int32_t *perm, *tok_item, *tok_win, *cmp_start, *slc_start, *win_start, *cmp_slc, *cmp_batch, *slc_batch,
      *item_start;
  int N, Nc, Ns, Nw, Hq, Hkv, hs, T, s_max;
  float scale, sl2;  // softmax scale, scale * log2(e)
  // sorted copies (bf16), row-major [rows][Hkv][D]: token K, V and pooled K, V
  const bf16_t *Ks, *Vs, *Kc, *Vc;
};
