// Generic SSA path: fp32 arithmetic (fp32 matrix instructions), any head_dim <= 128 (multiple of 8) and any head grouping up
// to 64 query heads per KV head.  Serves SSA_F32 problems and every shape the bf16 MFMA kernels do not cover.  Same
// mathematics as the MFMA path (paper eq. (2)-(6), Algorithm 1, window paragraph).
//
// One 16 x 16 tile of v_mfma_f32_16x16x4_f32 (A: lane l gives row l & 15, contraction index l >> 4; B: column l & 15, the
// same index; C: column l & 15, rows 4*(l >> 4) .. +3; "n" = l & 15, "quad" = l >> 4) is 16 keys x 16 query columns, the
// columns being (token, head) pairs of one KV head.  The index order inside a contraction is free, which removes every
// data movement between the two products of a tile:
//   * scores: step (s, i) contracts dims 16*s + 4*quad + i, so a lane's share of a row is DT 16-byte pieces;
//   * the next product contracts over keys, step i over keys 4*quad + i: exactly the four scores a lane holds, and the other
//     operand is DT consecutive dims (n*DT ..) of row 4*quad + i, one vector load; result row r of block b is dim r*DT + b.
// Operands come straight from memory (one KV head's rows stay in the caches), with the next tile's in flight during a
// tile; there is no LDS staging and no barrier inside a walk.  The wavefronts of a workgroup share their 16 columns (or
// 16 keys) and deal the tiles of the walk out among them, so that a problem of a few thousand rows fills the chip; their
// partial results meet in LDS and are added in wavefront order (every sum in one fixed order: no atomics).
// Bound: latency of the walks at a few thousand tokens (2874 tokens, 4 heads of 32, forward + backward: 6.55 -> 0.27 ms;
// the former kernels ran one row per wavefront with the dims in a scalar loop), fp32 matrix rate above (6000 tokens, 16 heads of
// 64: 35-60 of the 153 TFLOP/s a large fp32 product reaches).
#include "ssa_internal.h"
#include "profile.h"
#include "topk_device.h"
#include "mfma_launch.h"

#include <mutex>

namespace {

constexpr int WAVE = 64;
constexpr int NW = 4;        // wavefronts of the query-centric kernels
// wavefronts of the key-centric kernel (its operands of 128 dims want the registers of one wavefront per SIMD)
template <int DT> constexpr int nw_key() { return DT == 8 ? 4 : 8; }
constexpr float LOG2E_F = 1.4426950408889634f, LN2_F = 0.6931471805599453f;

typedef __attribute__((ext_vector_type(4))) float f4;

struct BlkView {
  const int32_t *perm, *tok_item, *tok_cmp, *tok_slc, *tok_win, *cmp_start, *slc_start, *win_start, *slc_child_start, *cmp_slc,
      *cmp_batch, *slc_batch, *item_start;
  int N, B, Nc, Ns;
};

static BlkView view_of(const ssa_blocks *b) {
  return BlkView{b->perm, b->tok_item, b->tok_cmp, b->tok_slc, b->tok_win, b->cmp_start, b->slc_start, b->win_start,
                 b->slc_child_start, b->cmp_slc, b->cmp_batch, b->slc_batch, b->item_start, b->N, b->B, b->Nc, b->Ns};
}

__device__ inline f4 mfma4(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

__device__ inline f4 ld4(const float *p) { return *reinterpret_cast<const f4 *>(p); }
__device__ inline f4 ld4(const uint16_t *p) {
  const uint2 w = *reinterpret_cast<const uint2 *>(p);
  return f4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xFFFF0000u), __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xFFFF0000u)};
}
__device__ inline void st4(float *p, f4 v) { *reinterpret_cast<f4 *>(p) = v; }
__device__ inline void st4(uint16_t *p, f4 v) {
  *reinterpret_cast<ushort4 *>(p) = make_ushort4(f32_to_bf16(v[0]), f32_to_bf16(v[1]), f32_to_bf16(v[2]), f32_to_bf16(v[3]));
}

// DT consecutive elements (DT = 1, 2, 4, 8) from an address aligned to their size.
template <int DT, typename T>
__device__ inline void ld_chunk(const T *p, float (&o)[DT]) {
  struct alignas(DT * sizeof(T) < 16 ? DT * sizeof(T) : 16) C { T v[DT]; };
  const C c = *reinterpret_cast<const C *>(p);
#pragma unroll
  for (int b = 0; b < DT; ++b) o[b] = io<T>::ld(c.v + b);
}
template <int DT, typename T>
__device__ inline void st_chunk(T *p, const float (&o)[DT]) {
  struct alignas(DT * sizeof(T) < 16 ? DT * sizeof(T) : 16) C { T v[DT]; };
  C c;
#pragma unroll
  for (int b = 0; b < DT; ++b) io<T>::st(c.v + b, o[b]);
  *reinterpret_cast<C *>(p) = c;
}

// A lane's 4*DT consecutive result dims (acc[b][i]: dim 4*DT*quad + i*DT + b of column n) to or from a row of floats.
template <int DT>
__device__ inline void acc_put(float *row, const f4 (&acc)[DT], int d = 16 * DT) {
  const int quad = threadIdx.x >> 4 & 3;
#pragma unroll
  for (int w = 0; w < DT; ++w) {
    f4 x;
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = acc[(4 * w + j) % DT][(4 * w + j) / DT];
    if (4 * DT * quad + 4 * w < d) st4(row + 4 * DT * quad + 4 * w, x);
  }
}
template <int DT>
__device__ inline void acc_add(const float *row, f4 (&acc)[DT]) {
  const int quad = threadIdx.x >> 4 & 3;
#pragma unroll
  for (int w = 0; w < DT; ++w) {
    const f4 x = ld4(row + 4 * DT * quad + 4 * w);
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[(4 * w + j) % DT][(4 * w + j) / DT] += x[j];
  }
}

// Reductions over the four quads of a column (lanes 16 apart), result in all of them.
__device__ inline float quad_sum(float v) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}
__device__ inline float quad_max(float v) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ inline int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }  // in a scalar register
__device__ inline unsigned wave_min_u(unsigned v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = min(v, (unsigned)__shfl_xor((int)v, off));
  return v;
}
__device__ inline int wave_max_i32(int v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = max(v, __shfl_xor(v, off));
  return v;
}

// Sorted fp32 copies of K,V and their per-compression-block means (eq. (5), mean pool over active tokens).  One workgroup
// per compression block; thread t keeps the 4 elements t % C of tokens t / C, t / C + 256 / C, ... (C = pieces of a row, at
// most 256), whose sums meet in LDS in thread order.
template <typename T>
__global__ __launch_bounds__(256) void g_sort_pool(const T *__restrict__ K, const T *__restrict__ V, BlkView bv, int row /*Hkv*d*/,
                                                   float *__restrict__ Ks, float *__restrict__ Vs, float *__restrict__ Kc,
                                                   float *__restrict__ Vc, uint32_t *ticket) {
  __shared__ f4 part[2][256];
  const int c = blockIdx.x;
  if (ticket && c == 0 && threadIdx.x == 0) *ticket = 0u;  // counter of the selection index's first pass
  const int b = bv.cmp_start[c], e = bv.cmp_start[c + 1];
  const float inv = 1.0f / (float)(e - b);
  const int c4 = row / 4, C = min(c4, 256), ngrp = 256 / C, grp = threadIdx.x / C;
  for (int f0 = 0; f0 < c4; f0 += C) {
    const int f = f0 + (int)threadIdx.x % C;
    f4 sk = {0.f, 0.f, 0.f, 0.f}, sv = sk;
    if (grp < ngrp && f < c4)
#pragma unroll 2
      for (int pos = b + grp; pos < e; pos += ngrp) {
        const size_t src = (size_t)bv.perm[pos] * row + 4 * f, dst = (size_t)pos * row + 4 * f;
        const f4 kk = ld4(K + src), vv = ld4(V + src);
        st4(Ks + dst, kk);
        st4(Vs + dst, vv);
        sk += kk;
        sv += vv;
      }
    part[0][threadIdx.x] = sk;
    part[1][threadIdx.x] = sv;
    __syncthreads();
    if ((int)threadIdx.x < C && f < c4) {
      for (int gi = 1; gi < ngrp; ++gi) { sk += part[0][gi * C + threadIdx.x]; sv += part[1][gi * C + threadIdx.x]; }
      f4 ok, ov;
#pragma unroll
      for (int i = 0; i < 4; ++i) { ok[i] = io<T>::round(sk[i] * inv); ov[i] = io<T>::round(sv[i] * inv); }
      st4(Kc + (size_t)c * row + 4 * f, ok);
      st4(Vc + (size_t)c * row + 4 * f, ov);
    }
    __syncthreads();
  }
}

// The 16 query columns of a workgroup: with h_s <= 16 heads per KV head, tpt tokens x h_s heads (columns past tpt*h_s are
// unused); with more heads, one token's heads 16 at a time.
struct Cols {
  int tok, h, pos, slot;
  bool valid;
};
__host__ __device__ inline int tokens_per_tile(int hs) { return hs <= 16 ? 16 / hs : 1; }
__host__ __device__ inline int tiles_per_token(int hs) { return hs <= 16 ? 1 : (hs + 15) / 16; }
__device__ inline Cols columns(const BlkView &bv, int hs, int g, int tile) {
  const int n = threadIdx.x & 15;
  Cols c;
  if (hs <= 16) {
    const int tpt = 16 / hs;
    c.slot = n / hs;
    c.pos = tile * tpt + c.slot;
    c.h = g * hs + n % hs;
    c.valid = c.slot < tpt && c.pos < bv.N;
  } else {
    const int ct = (hs + 15) / 16, hh = (tile % ct) * 16 + n;
    c.slot = 0;
    c.pos = tile / ct;
    c.h = g * hs + hh;
    c.valid = hh < hs;
  }
  if (!c.valid) { c.pos = 0; c.h = g * hs; }
  c.tok = bv.perm[c.pos];
  return c;
}

// A lane's share of one row as a score operand: dims 16*s + 4*quad .. +3, s < DT; zero past d and for a missing row.
template <typename T, int DT>
__device__ inline void ld_row(const T *row, int d, bool valid, f4 (&o)[DT], int quad) {
#pragma unroll
  for (int s = 0; s < DT; ++s) {
    const int dim = 16 * s + 4 * quad;
    o[s] = valid && dim < d ? ld4(row + dim) : f4{0.f, 0.f, 0.f, 0.f};
  }
}
template <typename T, int DT>
__device__ inline void ld_row(const T *row, int d, bool valid, f4 (&o)[DT]) { ld_row<T, DT>(row, d, valid, o, threadIdx.x >> 4 & 3); }
// The same for key rows, where finite garbage past d is harmless (it meets the zeros of the other operand): no selects.
template <int DT>
__device__ inline void ld_key(const float *row, int d, f4 (&o)[DT]) {
  const int quad = threadIdx.x >> 4 & 3;
#pragma unroll
  for (int s = 0; s < DT; ++s) o[s] = ld4(row + (16 * s + 4 * quad < d ? 16 * s + 4 * quad : 0));
}

template <int DT>
__device__ inline f4 dot16(const f4 (&a)[DT], const f4 (&b)[DT]) {
  f4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
#pragma unroll
  for (int s = 0; s < DT; ++s)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i & 1) c1 = mfma4(a[s][i], b[s][i], c1);
      else c0 = mfma4(a[s][i], b[s][i], c0);
    }
  return c0 + c1;
}

// Infinities and NaN.  A tile multiplies every key with every column, and the zero weight of a key that a column may not see
// does not cancel a non-finite element of that key.  Such an element leaves a non-finite sum, so a walk that ends with one is
// repeated one key at a time (the *_alone functions), each key added only to the columns that see it: what a row does not
// attend to never reaches it (a NaN of one batch item stays in that item), nor does a row's own element through padding.  A walk over finite data pays one look at its
// sums.  The repeated walks are written for few registers, not for speed.
template <int DT>
__device__ inline bool finite_sums(const f4 (&acc)[DT]) {
  unsigned most = 0u;
#pragma unroll
  for (int b = 0; b < DT; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i) most = max(most, __float_as_uint(acc[b][i]) & 0x7FFFFFFFu);
  asm volatile("" : "+v"(most));  // (the comparison stays one of integers: this file is compiled as if NaN did not occur)
  return most < 0x7F800000u;
}
// The thread's number, hidden from the compiler: what a repeated walk derives from it is not kept in registers from the start.
__device__ inline int thread_again() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}
// Element `row` (of 16, uniform) of lane n's column, from the lane that holds it (w: rows 4*quad .. +3 of column n).
__device__ inline float of_row(const f4 &w, int row) {
  const float x = row & 2 ? (row & 1 ? w[3] : w[2]) : (row & 1 ? w[1] : w[0]);
  return __shfl(x, (int)(threadIdx.x & 15) + 16 * (row >> 2));
}
// acc += row * w for one row of the other operand (lane n's DT elements of it at p), in the columns with `mine`.
template <int DT, typename T>
__device__ inline void add_alone(f4 (&acc)[DT], const T *p, float w, bool mine) {
  const bool first = (threadIdx.x & 48) == 0;  // the row is index 0 of the contraction
  float x[DT];
  ld_chunk<DT>(p, x);
#pragma unroll
  for (int b = 0; b < DT; ++b) {
    const f4 r = mfma4(first ? x[b] : 0.f, first ? w : 0.f, acc[b]);
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[b][i] = mine ? r[i] : acc[b][i];
  }
}

// Walks: next() moves to this wavefront's next 16-key tile.  kb: its first key; last: the last existing key of its range;
// lo, hi: the keys this lane's column may see.
struct RangeWalk {  // one range [k0, k1) for all columns, with a window of its own per column
  int kb, k1, lo, hi, last, step;
  __device__ RangeWalk(int k0, int k1_, int lo_, int hi_, int wid, int nw)
      : kb(k0 + 16 * (wid - nw)), k1(k1_), lo(lo_), hi(hi_), last(k1_ - 1), step(16 * nw) {}
  __device__ bool next() { kb += step; return kb < k1; }
};
// The union of the selected blocks of a workgroup's tokens, ascending, in LDS: keys [k0, k1) of the block and a bit per
// token that selected it.
struct UnionEntry { int k0, k1; unsigned tokens; };
struct UnionWalk {
  const UnionEntry *u, *end;
  int kb, kend, lo, hi, last, step, wid, nw, phase;
  unsigned bit;  // this lane's column: 1 << token slot, 0 for an unused column
  __device__ UnionWalk(const UnionEntry *u_, int count, int slot, bool valid, int wid_, int nw_)
      : u(u_), end(u_ + count), kb(0), kend(0), lo(0), hi(0), last(0), step(16 * nw_), wid(wid_), nw(nw_), phase(0),
        bit(valid ? 1u << slot : 0u) {}
  __device__ bool next() {
    kb += step;
    while (kb >= kend) {
      if (u == end) return false;
      const int k0 = __builtin_amdgcn_readfirstlane(u->k0);
      kend = __builtin_amdgcn_readfirstlane(u->k1);
      const bool on = (u->tokens & bit) != 0;
      ++u;
      last = kend - 1;
      lo = on ? k0 : 0;
      hi = on ? kend : 0;
      kb = k0 + 16 * ((wid - phase + nw) % nw);
      phase = (phase + (kend - k0 + 15) / 16) % nw;
    }
    return true;
  }
};

// Builds the union of the selected blocks of tokens pos0 .. pos0+ntok-1 (rows of I in any order, invalid ids ignored).
// LDS: raw [ntok*T], first [ntok*T], u [ntok*T]; returns the number of entries.
__host__ __device__ inline size_t union_lds_bytes(int ntok, int T) { return (size_t)ntok * T * (sizeof(UnionEntry) + 8); }
__device__ inline int build_union(const BlkView &bv, const int32_t *idx, int Hkv, int T, int g, int pos0, int ntok, int cap,
                                  unsigned *smem, UnionEntry *&u) {
  unsigned *raw = smem, *first = raw + cap;
  u = (UnionEntry *)(first + cap);
  const int n = ntok * T;
  for (int e = threadIdx.x; e < n; e += blockDim.x) {
    const int t = e / T, b = idx[((size_t)bv.perm[pos0 + t] * Hkv + g) * T + e % T];
    raw[e] = b >= 0 && b < bv.Ns ? (unsigned)b : ~0u;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < n; e += blockDim.x) {
    const unsigned v = raw[e];
    bool f = v != ~0u;
    for (int i = 0; i < e; ++i) f = f && raw[i] != v;
    first[e] = f ? 1u : 0u;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < n; e += blockDim.x) {
    if (!first[e]) continue;
    const unsigned v = raw[e];
    unsigned tokens = 0u;
    int r = 0;
    for (int t = 0, i = 0; t < ntok; ++t)
      for (int j = 0; j < T; ++j, ++i) {
        if (raw[i] == v) tokens |= 1u << t;
        r += raw[i] < v ? (int)first[i] : 0;
      }
    u[r] = UnionEntry{bv.slc_start[v], bv.slc_start[v + 1], tokens};
  }
  int total = 0;
  for (int i = threadIdx.x & 63; i < n; i += WAVE) total += (int)first[i];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) total += __shfl_xor(total, off);
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(total);
}

// ---- forward ------------------------------------------------------------------------------------------------------------
template <int DT>
struct FwdTile {
  f4 k[DT];
  float vt[4][DT];
};
template <int DT>
__device__ inline void ld_fwd_tile(FwdTile<DT> &t, const float *Kg, const float *Vg, int stride, int d, int kb, int last) {
  const int n = threadIdx.x & 15, quad = threadIdx.x >> 4 & 3, c = n * DT < d ? n * DT : 0;
  ld_key<DT>(Kg + (size_t)min(kb + n, last) * stride, d, t.k);
#pragma unroll
  for (int i = 0; i < 4; ++i) ld_chunk<DT>(Vg + (size_t)min(kb + 4 * quad + i, last) * stride + c, t.vt[i]);
}

template <int DT>
struct State {
  f4 o[DT];
  float m, l;  // reference maximum (log2 units) of the column; this lane's share of the sum
};

template <int DT>
__device__ inline void clear(State<DT> &st) {
  st.m = -INFINITY;
  st.l = 0.f;
#pragma unroll
  for (int b = 0; b < DT; ++b) st.o[b] = f4{0.f, 0.f, 0.f, 0.f};
}
// Scores of one tile (masked: the column sees keys rel .. rel + 3 inside [0, len)) to probabilities, the reference raised where needed.
template <int DT>
__device__ inline void softmax_reference(State<DT> &st, f4 &v, int rel, int len, float sl2) {
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = (unsigned)(rel + i) < (unsigned)len ? v[i] * sl2 : -INFINITY;
  const float pm = fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
  if (__any(pm > st.m + 8.f)) {
    const float mn = fmaxf(st.m, quad_max(pm));
    const float alpha = mn == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(st.m - mn);
    st.m = mn;
    st.l *= alpha;
#pragma unroll
    for (int b = 0; b < DT; ++b) st.o[b] *= alpha;
  }
}
template <int DT>
__device__ inline f4 softmax_step(State<DT> &st, f4 v, int rel, int len, float sl2) {
  softmax_reference(st, v, rel, len, sl2);
  const float neg = st.m == -INFINITY ? -INFINITY : -st.m;
  f4 p;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    p[i] = __builtin_amdgcn_exp2f(v[i] + neg);
    st.l += p[i];
  }
  return p;
}

template <int DT, class Walk>
__device__ inline void attend_alone(State<DT> &st, const f4 (&q)[DT], Walk w, const float *Kg, const float *Vg, int stride, int d, float sl2) {
  const int t = thread_again(), n = t & 15, quad = t >> 4 & 3, c = n * DT < d ? n * DT : 0;
  clear(st);
#pragma unroll 1
  while (w.next()) {
    f4 k[DT];
    ld_row<float, DT>(Kg + (size_t)min(w.kb + n, w.last) * stride, d, true, k, quad);
    const f4 p = softmax_step(st, dot16<DT>(k, q), w.kb + 4 * quad - w.lo, w.hi - w.lo, sl2);
#pragma unroll 1
    for (int key = 0; key < 16; ++key)
      add_alone<DT>(st.o, Vg + (size_t)min(w.kb + key, w.last) * stride + c, of_row(p, key), (unsigned)(w.kb + key - w.lo) < (unsigned)(w.hi - w.lo));
  }
}

// Softmax attention of the 16 columns over a walk (Algorithm 1's inner loop).  The reference maximum is raised lazily: a
// column's exponents stay below 2^8, and the result does not depend on the reference.
template <int DT, class Walk>
__device__ inline void attend(State<DT> &st, const f4 (&q)[DT], Walk w, const float *Kg, const float *Vg, int stride, int d, float sl2) {
  const int quad = threadIdx.x >> 4 & 3;
  const Walk again = w;
  clear(st);
  bool more = w.next();
  FwdTile<DT> cur, nxt;
  if (more) ld_fwd_tile(cur, Kg, Vg, stride, d, w.kb, w.last);
  while (more) {
    const int rel = w.kb + 4 * quad - w.lo, len = w.hi - w.lo;
    more = w.next();
    if (more) ld_fwd_tile(nxt, Kg, Vg, stride, d, w.kb, w.last);
    f4 v = dot16<DT>(cur.k, q);
    softmax_reference(st, v, rel, len, sl2);
    const float neg = st.m == -INFINITY ? -INFINITY : -st.m;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float p = __builtin_amdgcn_exp2f(v[i] + neg);
      st.l += p;
#pragma unroll
      for (int b = 0; b < DT; ++b) st.o[b] = mfma4(cur.vt[i][b], p, st.o[b]);
    }
    cur = nxt;
  }
  if (__builtin_expect(!__all(finite_sums<DT>(st.o)), 0)) attend_alone<DT>(st, q, again, Kg, Vg, stride, d, sl2);
}

// Merge of the wavefronts' states through LDS: thread t gets column t / 16, dims (t % 16)*DT .. +DT-1, normalised, and the
// column's log-sum-exp (natural).
template <int DT>
struct MergeBuf {
  float ml[NW][16][2];
  float o[NW][16][16 * DT + 4];
};
template <int DT>
__device__ inline float merge_waves(MergeBuf<DT> &mb, const State<DT> &st, float (&o)[DT]) {
  const int wid = threadIdx.x >> 6, n = threadIdx.x & 15, quad = threadIdx.x >> 4 & 3;
  const float l = quad_sum(st.l);
  __syncthreads();  // the buffer may still be read from the merge before
  if (quad == 0) { mb.ml[wid][n][0] = st.m; mb.ml[wid][n][1] = l; }
  acc_put<DT>(mb.o[wid][n], st.o);
  __syncthreads();
  const int col = threadIdx.x >> 4, c = (threadIdx.x & 15) * DT;
  float M = -INFINITY, L = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) M = fmaxf(M, mb.ml[w][col][0]);
#pragma unroll
  for (int b = 0; b < DT; ++b) o[b] = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const float mw = mb.ml[w][col][0], f = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - M);
    L += f * mb.ml[w][col][1];
#pragma unroll
    for (int b = 0; b < DT; ++b) o[b] += f * mb.o[w][col][c + b];
  }
  const float inv = L > 0.f ? 1.0f / L : 0.f;
#pragma unroll
  for (int b = 0; b < DT; ++b) o[b] *= inv;
  return L > 0.f ? M * LN2_F + __logf(L) : -INFINITY;
}

struct FwdArgs {
  const void *Q, *gates;
  BlkView bv;
  const int32_t *idx;
  int Hq, Hkv, hs, d, T;
  float sl2;
  const float *K, *V;    // cmp kernel: pooled rows; selection + window kernel: token rows
  void *Ob, *out;
  float *lse;
};

// Bounds [lo, hi) of the union over valid columns.
__device__ inline void union_range(int lo, int hi, bool valid, int &k0, int &k1) {
  k0 = (int)__builtin_amdgcn_readfirstlane((int)wave_min_u(valid ? (unsigned)lo : 0x7fffffffu));
  k1 = __builtin_amdgcn_readfirstlane(wave_max_i32(valid ? hi : 0));
  if (k1 <= k0) k0 = k1 = 0;
}

// Compression branch: one workgroup per 16 columns.  (The repeated walk's code would cost the kernel a wavefront per SIMD; the
// bound keeps it at what the tile loop takes.)
template <typename T, int DT>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(DT == 2 ? 6 : DT == 4 ? 4 : 1))) void g_cmp_fwd(FwdArgs a) {
  __shared__ MergeBuf<DT> mb;
  __shared__ int scol[16];
  const int g = blockIdx.y, wid = wave_id();
  const Cols c = columns(a.bv, a.hs, g, blockIdx.x);
  if (threadIdx.x < 16) scol[threadIdx.x] = c.valid ? c.tok * a.Hq + c.h : -1;
  const int item = a.bv.tok_item[c.pos], lo = c.valid ? a.bv.cmp_batch[item] : 0, hi = c.valid ? a.bv.cmp_batch[item + 1] : 0;
  int k0, k1;
  union_range(lo, hi, c.valid, k0, k1);
  f4 q[DT];
  ld_row<T, DT>((const T *)a.Q + ((size_t)c.tok * a.Hq + c.h) * a.d, a.d, c.valid, q);
  State<DT> st;
  attend<DT>(st, q, RangeWalk(k0, k1, lo, hi, wid, NW), a.K + g * a.d, a.V + g * a.d, a.Hkv * a.d, a.d, a.sl2);
  float o[DT];
  const float lse = merge_waves<DT>(mb, st, o);
  const int th = scol[threadIdx.x >> 4], ch = (threadIdx.x & 15) * DT;
  if (th < 0) return;
  if (ch < a.d) st_chunk<DT>((T *)a.Ob + (size_t)th * a.d + ch, o);
  if (ch == 0) a.lse[th] = lse;
}

// Window branch, selection branch and the gated sum of eq. (4): one workgroup per 16 columns.
template <typename T, int DT>
__global__ __launch_bounds__(64 * NW) void g_slc_win_fwd(FwdArgs a) {
  extern __shared__ unsigned ids[];  // build_union
  __shared__ MergeBuf<DT> mb;
  __shared__ int scol[16];
  const int g = blockIdx.y, wid = wave_id(), stride = a.Hkv * a.d;
  const Cols c = columns(a.bv, a.hs, g, blockIdx.x);
  if (threadIdx.x < 16) scol[threadIdx.x] = c.valid ? c.tok * a.Hq + c.h : -1;
  const int tpt = tokens_per_tile(a.hs), pos0 = (int)blockIdx.x / tiles_per_token(a.hs) * tpt;
  UnionEntry *un;
  const int n_un = build_union(a.bv, a.idx, a.Hkv, a.T, g, pos0, min(tpt, a.bv.N - pos0), tpt * a.T, ids, un);
  f4 q[DT];
  ld_row<T, DT>((const T *)a.Q + ((size_t)c.tok * a.Hq + c.h) * a.d, a.d, c.valid, q);
  const float *Kg = a.K + g * a.d, *Vg = a.V + g * a.d;
  const int win = a.bv.tok_win[c.pos], lo = c.valid ? a.bv.win_start[win] : 0, hi = c.valid ? a.bv.win_start[win + 1] : 0;
  int k0, k1;
  union_range(lo, hi, c.valid, k0, k1);
  State<DT> st;
  float ow[DT], os[DT];
  attend<DT>(st, q, RangeWalk(k0, k1, lo, hi, wid, NW), Kg, Vg, stride, a.d, a.sl2);
  const float lse_w = merge_waves<DT>(mb, st, ow);
  attend<DT>(st, q, UnionWalk(un, n_un, c.slot, c.valid, wid, NW), Kg, Vg, stride, a.d, a.sl2);
  const float lse_s = merge_waves<DT>(mb, st, os);
  const int th = scol[threadIdx.x >> 4], ch = (threadIdx.x & 15) * DT;
  if (th < 0) return;
  const size_t NH = (size_t)a.bv.N * a.Hq;
  if (ch == 0) { a.lse[NH + th] = lse_s; a.lse[2 * NH + th] = lse_w; }
  if (ch >= a.d) return;
  T *Ob = (T *)a.Ob;
  const size_t off = (size_t)th * a.d + ch;
  st_chunk<DT>(Ob + NH * a.d + off, os);
  st_chunk<DT>(Ob + 2 * NH * a.d + off, ow);
  float oc[DT], r[DT];
  ld_chunk<DT>(Ob + off, oc);
  const T *gt = (const T *)a.gates + (size_t)th * 3;
  const float w0 = io<T>::ld(gt), w1 = io<T>::ld(gt + 1), w2 = io<T>::ld(gt + 2);
#pragma unroll
  for (int b = 0; b < DT; ++b) r[b] = w0 * oc[b] + w1 * io<T>::round(os[b]) + w2 * io<T>::round(ow[b]);
  st_chunk<DT>((T *)a.out + off, r);
}

// Selection scores (eq. (6)) and top-k.  One workgroup per tw tokens of one KV head: chunks of KC pooled keys, their
// probabilities in LDS per column, then one thread per (token, selection block) adds its children's probabilities head by
// head in a fixed order.
constexpr int KC = 256;
struct ScoreArgs {
  const void *Q;
  BlkView bv;
  const float *Kc, *lse;  // lse: compression branch [N,Hq], caller order
  int32_t *idx;
  int Hq, Hkv, hs, d, T, tw, s_max;
  float sl2;
};
size_t score_lds_bytes(int tw, int s_max) { return ((size_t)16 * (KC + 4) + (size_t)tw * s_max + (size_t)NW * ((s_max + 31) / 32)) * 4; }

template <typename T, int DT>
__global__ __launch_bounds__(64 * NW) void g_scores_topk(ScoreArgs a) {
  extern __shared__ float sm[];
  float *P = sm, *S = P + 16 * (KC + 4);  // P [16 columns][KC + 4], S [tw][s_max]
  uint32_t *marks = (uint32_t *)(S + (size_t)a.tw * a.s_max);
  const int g = blockIdx.y, wid = wave_id(), n = threadIdx.x & 15, quad = threadIdx.x >> 4 & 3;
  const int pos0 = blockIdx.x * a.tw, ntok = min(a.tw, a.bv.N - pos0), hc = min(a.hs, 16), cts = tiles_per_token(a.hs);
  for (int i = threadIdx.x; i < a.tw * a.s_max; i += 64 * NW) S[i] = 0.f;
  const int i0 = a.bv.tok_item[pos0], i1 = a.bv.tok_item[pos0 + ntok - 1];
  const int k0 = a.bv.cmp_batch[i0], k1 = a.bv.cmp_batch[i1 + 1];
  for (int kc = k0; kc < k1; kc += KC) {
    const int ke = min(kc + KC, k1), b0 = a.bv.cmp_slc[kc], nb = a.bv.cmp_slc[ke - 1] + 1 - b0;
    for (int ct = 0; ct < cts; ++ct) {
      const int slot = cts == 1 ? n / hc : 0, head = cts == 1 ? n % hc : ct * 16 + n;
      const bool valid = slot < ntok && head < a.hs;
      const size_t th = (size_t)a.bv.perm[pos0 + (valid ? slot : 0)] * a.Hq + g * a.hs + (valid ? head : 0);
      f4 q[DT];
      ld_row<T, DT>((const T *)a.Q + th * a.d, a.d, valid, q);
      const float nl = valid ? -a.lse[th] * LOG2E_F : -INFINITY;
      for (int kb = kc + 16 * wid; kb < ke; kb += 16 * NW) {
        f4 k[DT];
        ld_row<float, DT>(a.Kc + ((size_t)min(kb + n, k1 - 1) * a.Hkv + g) * a.d, a.d, true, k);
        const f4 v = dot16<DT>(k, q);
        f4 p;
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(v[i], a.sl2, nl));
        st4(P + n * (KC + 4) + kb - kc + 4 * quad, p);
      }
      __syncthreads();
      const int nh = cts == 1 ? a.hs : min(16, a.hs - ct * 16);
      for (int e = threadIdx.x; e < ntok * nb; e += 64 * NW) {
        const int sl = e / nb, b = b0 + e % nb, item = a.bv.tok_item[pos0 + sl], s0 = a.bv.slc_batch[item];
        if (b < s0 || b >= a.bv.slc_batch[item + 1]) continue;
        const int c0 = max(a.bv.slc_child_start[b], kc), c1 = min(a.bv.slc_child_start[b + 1], ke);
        float acc = S[(size_t)sl * a.s_max + b - s0];
        for (int c = c0; c < c1; ++c)
          for (int hl = 0; hl < nh; ++hl) acc += P[(sl * nh * (cts == 1) + hl) * (KC + 4) + c - kc];
        S[(size_t)sl * a.s_max + b - s0] = acc;
      }
      __syncthreads();
    }
  }
  for (int sl = wid; sl < ntok; sl += NW) {
    const int item = a.bv.tok_item[pos0 + sl], s0 = a.bv.slc_batch[item], cnt = a.bv.slc_batch[item + 1] - s0;
    topk_wave(S + (size_t)sl * a.s_max, cnt, a.T, s0, a.idx + ((size_t)a.bv.perm[pos0 + sl] * a.Hkv + g) * a.T, marks + wid * ((a.s_max + 31) / 32));
  }
}

__global__ void g_topk_from_scores(const float *__restrict__ scores, BlkView bv, int Hkv, int Tk, int s_max,
                                   const int32_t *__restrict__ inv_perm, int32_t *__restrict__ idx) {
  extern __shared__ float smem[];
  float *S = smem;
  uint32_t *sel = (uint32_t *)(S + s_max);
  const int tok = blockIdx.x / Hkv, g = blockIdx.x % Hkv;
  const int item = bv.tok_item[inv_perm[tok]];
  const int s0 = bv.slc_batch[item], n = bv.slc_batch[item + 1] - s0;
  for (int i = threadIdx.x; i < n; i += WAVE) S[i] = scores[((size_t)tok * Hkv + g) * s_max + i];
  __syncthreads();
  topk_wave(S, n, Tk, s0, idx + ((size_t)tok * Hkv + g) * Tk, sel);
}

// ---- backward -----------------------------------------------------------------------------------------------------------
// Per (query row, key) pair of branch b with gate w: P = exp(S - lse), dS = P (w <dO, V> - delta) scale, delta = w <dO, O_b>;
// dV += w P dO, dQ += dS K, dK += dS Q.
template <int DT>
struct DqTile {
  f4 k[DT], v[DT];
  float kt[4][DT];
};
template <int DT>
__device__ inline void ld_dq_tile(DqTile<DT> &t, const float *Kg, const float *Vg, int stride, int d, int kb, int last) {
  const int n = threadIdx.x & 15, quad = threadIdx.x >> 4 & 3, c = n * DT < d ? n * DT : 0;
  const size_t r = (size_t)min(kb + n, last) * stride;
  ld_key<DT>(Kg + r, d, t.k);
  ld_key<DT>(Vg + r, d, t.v);
#pragma unroll
  for (int i = 0; i < 4; ++i) ld_chunk<DT>(Kg + (size_t)min(kb + 4 * quad + i, last) * stride + c, t.kt[i]);
}

struct RowInfo { float lse2, delta, w; };

template <int DT, class Walk>
__device__ inline void attend_bwd(f4 (&dq)[DT], const f4 (&q)[DT], const f4 (&go)[DT], const RowInfo &ri, Walk w, const float *Kg,
                                  const float *Vg, int stride, int d, float sl2, float scale) {
  const int quad = threadIdx.x >> 4 & 3;
  bool more = w.next();
  DqTile<DT> cur, nxt;
  if (more) ld_dq_tile(cur, Kg, Vg, stride, d, w.kb, w.last);
  while (more) {
    const int rel = w.kb + 4 * quad - w.lo, len = w.hi - w.lo;
    more = w.next();
    if (more) ld_dq_tile(nxt, Kg, Vg, stride, d, w.kb, w.last);
    const f4 s = dot16<DT>(cur.k, q), dp = dot16<DT>(cur.v, go);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float p = (unsigned)(rel + i) < (unsigned)len ? __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], sl2, -ri.lse2)) : 0.f;
      const float ds = p * (ri.w * dp[i] - ri.delta) * scale;
#pragma unroll
      for (int b = 0; b < DT; ++b) dq[b] = mfma4(cur.kt[i][b], ds, dq[b]);
    }
    cur = nxt;
  }
}

template <int DT, class Walk>
__device__ inline void attend_bwd_alone(f4 (&dq)[DT], const f4 (&q)[DT], const f4 (&go)[DT], const RowInfo &ri, Walk w, const float *Kg,
                                        const float *Vg, int stride, int d, float sl2, float scale) {
  const int t = thread_again(), n = t & 15, quad = t >> 4 & 3, c = n * DT < d ? n * DT : 0;
#pragma unroll 1
  while (w.next()) {
    const size_t r = (size_t)min(w.kb + n, w.last) * stride;
    f4 x[DT], ds;
    ld_row<float, DT>(Kg + r, d, true, x, quad);
    const f4 s = dot16<DT>(x, q);
    ld_row<float, DT>(Vg + r, d, true, x, quad);
    const f4 dp = dot16<DT>(x, go);
#pragma unroll
    for (int i = 0; i < 4; ++i) ds[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], sl2, -ri.lse2)) * (ri.w * dp[i] - ri.delta) * scale;
#pragma unroll 1
    for (int key = 0; key < 16; ++key)
      add_alone<DT>(dq, Kg + (size_t)min(w.kb + key, w.last) * stride + c, of_row(ds, key), (unsigned)(w.kb + key - w.lo) < (unsigned)(w.hi - w.lo));
  }
}

struct DqArgs {
  const void *Q, *dO, *Ob, *gates;
  BlkView bv;
  const int32_t *idx;
  int Hq, Hkv, hs, d, T;
  float scale, sl2;
  const float *Ks, *Vs, *Kc, *Vc, *lse;
  void *dQ, *dgates;
  f4 *info;  // [3][N*Hq]: lse (log2 units), delta, gate
};

// dgates, the row scalars and dQ of all three branches for 16 columns.
template <typename T, int DT>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(DT <= 2 ? 4 : 1))) void g_bwd_dq(DqArgs a) {
  extern __shared__ unsigned ids[];
  __shared__ float part[NW][16][16 * DT + 4];
  __shared__ int scol[16];
  const int g = blockIdx.y, wid = wave_id(), n = threadIdx.x & 15, quad = threadIdx.x >> 4 & 3, stride = a.Hkv * a.d;
  const Cols c = columns(a.bv, a.hs, g, blockIdx.x);
  if (threadIdx.x < 16) scol[threadIdx.x] = c.valid ? c.tok * a.Hq + c.h : -1;
  const int tpt = tokens_per_tile(a.hs), pos0 = (int)blockIdx.x / tiles_per_token(a.hs) * tpt;
  UnionEntry *un;
  const int n_un = build_union(a.bv, a.idx, a.Hkv, a.T, g, pos0, min(tpt, a.bv.N - pos0), tpt * a.T, ids, un);
  const size_t th = (size_t)c.tok * a.Hq + c.h, NH = (size_t)a.bv.N * a.Hq;
  f4 q[DT], go[DT];
  ld_row<T, DT>((const T *)a.Q + th * a.d, a.d, c.valid, q);
  ld_row<T, DT>((const T *)a.dO + th * a.d, a.d, c.valid, go);
  RowInfo ri[3];
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    f4 ob[DT];
    ld_row<T, DT>((const T *)a.Ob + (b * NH + th) * a.d, a.d, c.valid, ob);
    float dot = 0.f;
#pragma unroll
    for (int s = 0; s < DT; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) dot += go[s][i] * ob[s][i];
    dot = quad_sum(dot);
    const float w = io<T>::ld((const T *)a.gates + th * 3 + b), l2 = a.lse[b * NH + th] * LOG2E_F;
    ri[b] = RowInfo{c.valid ? l2 : INFINITY, w * dot, w};
    if (wid == b && quad == 0 && c.valid) {  // (NW >= 3 wavefronts share the columns)
      io<T>::st((T *)a.dgates + th * 3 + b, dot);
      a.info[b * NH + th] = f4{l2, w * dot, w, 0.f};
    }
  }
  f4 dq[DT];
  const float *Kg = a.Ks + g * a.d, *Vg = a.Vs + g * a.d;
  auto walks = [&](auto alone) {
    auto one = [&](const RowInfo &r, auto w, const float *K, const float *V) {
      if constexpr (decltype(alone)::value) attend_bwd_alone<DT>(dq, q, go, r, w, K, V, stride, a.d, a.sl2, a.scale);
      else attend_bwd<DT>(dq, q, go, r, w, K, V, stride, a.d, a.sl2, a.scale);
    };
#pragma unroll
    for (int b = 0; b < DT; ++b) dq[b] = f4{0.f, 0.f, 0.f, 0.f};
    int k0, k1;
    {
      const int item = a.bv.tok_item[c.pos], lo = c.valid ? a.bv.cmp_batch[item] : 0, hi = c.valid ? a.bv.cmp_batch[item + 1] : 0;
      union_range(lo, hi, c.valid, k0, k1);
      one(ri[0], RangeWalk(k0, k1, lo, hi, wid, NW), a.Kc + g * a.d, a.Vc + g * a.d);
    }
    one(ri[1], UnionWalk(un, n_un, c.slot, c.valid, wid, NW), Kg, Vg);
    {
      const int win = a.bv.tok_win[c.pos], lo = c.valid ? a.bv.win_start[win] : 0, hi = c.valid ? a.bv.win_start[win + 1] : 0;
      union_range(lo, hi, c.valid, k0, k1);
      one(ri[2], RangeWalk(k0, k1, lo, hi, wid, NW), Kg, Vg);
    }
  };
  walks(std::false_type());
  if (__builtin_expect(!__all(finite_sums<DT>(dq)), 0)) walks(std::true_type());
  acc_put<DT>(part[wid][n], dq);
  __syncthreads();
  const int col = threadIdx.x >> 4, ch = (threadIdx.x & 15) * DT, to = scol[col];
  if (to < 0 || ch >= a.d) return;
  float r[DT];
#pragma unroll
  for (int b = 0; b < DT; ++b) {
    r[b] = part[0][col][ch + b];
#pragma unroll
    for (int w = 1; w < NW; ++w) r[b] += part[w][col][ch + b];
  }
  st_chunk<DT>((T *)a.dQ + (size_t)to * a.d + ch, r);
}

// dK, dV of 16 keys of one KV head: the query rows (token x head of the group) that attend to them in tiles of 16, dealt out
// to the wavefronts.  Three kinds of workgroup in one launch:
//   window:      16 consecutive sorted tokens; queries: the tokens of their windows;
//   selection:   16 tokens of one selection block; queries: a chunk of the block's selector list;
//   compression: 16 pooled keys; queries: one part of their items' tokens.
struct DkvArgs {
  const void *Q, *dO;
  BlkView bv;
  int Hq, Hkv, hs, d;
  float scale, sl2;
  const float *Ks, *Vs, *Kc, *Vc;
  const f4 *info;
  const int32_t *sel_list, *chunk_start, *part_row_start;  // lists of caller indices
  const ChunkRef *chunk_order;
  int slc_tiles, cmp_splits;
  long long n_win, n_slc;        // workgroups of the first two kinds
  long long first;               // number of this launch's first workgroup
  float *dKs, *dVs, *pK, *pV, *dKc, *dVc;  // window part [N][Hkv][d]; selection partials [rows][d]; [splits][Nc][Hkv][d]
};

template <typename T, int DT>
__global__ __launch_bounds__(64 * nw_key<DT>()) __attribute__((amdgpu_waves_per_eu(DT <= 2 ? 4 : 1))) void g_bwd_dkv(DkvArgs a) {
  constexpr int NW_KEY = nw_key<DT>();
  __shared__ float part[NW_KEY / 2][2][16][16 * DT + 4];
  const int wid = wave_id(), n = threadIdx.x & 15, quad = threadIdx.x >> 4 & 3, stride = a.Hkv * a.d;
  int g, branch, key0, kend, q0, q1, qlo, qhi;  // q: token indices (sorted positions, or places in the list)
  const int32_t *list = nullptr;
  const float *Kr = a.Ks, *Vr = a.Vs;
  float *oK, *oV;     // row of key0
  int ostride;
  const long long w0 = a.first + blockIdx.x, w1 = w0 - a.n_win;
  if (w1 < 0) {
    const int wg = (int)w0;
    branch = 2;
    g = wg % a.Hkv;
    key0 = wg / a.Hkv * 16;
    kend = a.bv.N;
    const int w = a.bv.tok_win[min(key0 + n, kend - 1)];
    qlo = a.bv.win_start[w];
    qhi = a.bv.win_start[w + 1];
    union_range(qlo, qhi, true, q0, q1);
    oK = a.dKs + (size_t)key0 * stride + g * a.d;
    oV = a.dVs + (size_t)key0 * stride + g * a.d;
    ostride = stride;
  } else if (w1 < a.n_slc) {
    branch = 1;
    const int ci = (int)(w1 / a.slc_tiles), tile = (int)(w1 % a.slc_tiles);
    if (ci >= a.chunk_start[a.Hkv * a.bv.Ns]) return;
    const ChunkRef cr = a.chunk_order[ci];
    g = cr.key / a.bv.Ns;
    const int blk = cr.key % a.bv.Ns, kbeg = a.bv.slc_start[blk];
    kend = a.bv.slc_start[blk + 1];
    key0 = kbeg + 16 * tile;
    if (key0 >= kend) return;
    list = a.sel_list;
    q0 = qlo = cr.first;
    q1 = qhi = cr.first + cr.count;
    const size_t row = (size_t)a.part_row_start[cr.key] + (size_t)cr.chunk * (kend - kbeg) + (key0 - kbeg);
    oK = a.pK + row * a.d;
    oV = a.pV + row * a.d;
    ostride = a.d;
  } else {
    int wg = (int)(w1 - a.n_slc);
    branch = 0;
    const int sp = wg % a.cmp_splits;
    wg /= a.cmp_splits;
    g = wg % a.Hkv;
    key0 = wg / a.Hkv * 16;
    kend = a.bv.Nc;
    const int item = a.bv.tok_item[a.bv.cmp_start[min(key0 + n, kend - 1)]];
    qlo = a.bv.item_start[item];
    qhi = a.bv.item_start[item + 1];
    union_range(qlo, qhi, true, q0, q1);
    const int per = (q1 - q0 + a.cmp_splits - 1) / a.cmp_splits;
    q0 = min(q1, q0 + sp * per);
    q1 = min(q1, q0 + per);
    Kr = a.Kc;
    Vr = a.Vc;
    oK = a.dKc + ((size_t)sp * a.bv.Nc + key0) * stride + g * a.d;
    oV = a.dVc + ((size_t)sp * a.bv.Nc + key0) * stride + g * a.d;
    ostride = stride;
  }
  const bool key_on = key0 + n < kend;
  f4 k[DT], v[DT];
  {
    const size_t r = (size_t)min(key0 + n, kend - 1) * stride + g * a.d;
    ld_row<float, DT>(Kr + r, a.d, key_on, k);
    ld_row<float, DT>(Vr + r, a.d, key_on, v);
  }
  f4 dk[DT], dv[DT];
#pragma unroll
  for (int b = 0; b < DT; ++b) dk[b] = dv[b] = f4{0.f, 0.f, 0.f, 0.f};
  const int ne = (q1 - q0) * a.hs;
  const f4 *info = a.info + (size_t)branch * a.bv.N * a.Hq;
  const T *Q = (const T *)a.Q, *dO = (const T *)a.dO;
  const int c = n * DT < a.d ? n * DT : 0;
  // element e of the walk: token q0 + e / h_s, head e % h_s.  A lane follows element 16*wid + n, + 16*NW_KEY, ... (token
  // and head advance by constants); th: its row of the caller's tensors, ql: its token index, both clamped past the end.
  const int dt_ = 16 * NW_KEY / a.hs, dh = 16 * NW_KEY - dt_ * a.hs;
  int tq = (16 * wid + n) / a.hs, hd = 16 * wid + n - tq * a.hs;
  auto row_of = [&](int t) { return (list ? list[t] : a.bv.perm[t]) * a.Hq + g * a.hs + hd; };
  int th = ne > 0 ? row_of(min(q0 + tq, q1 - 1)) : 0, ql = q0 + tq;
  for (int e0 = 16 * wid; e0 < ne; e0 += 16 * NW_KEY) {
    f4 qr[DT], gr[DT];
    const int rows = th, qls = ql;  // lane n's row; the rows 4*quad + i of the second product are those of lanes 4*quad + i
#pragma unroll
    for (int s = 0; s < DT; ++s) {
      const int dim = 16 * s + 4 * quad < a.d ? 16 * s + 4 * quad : 0;
      qr[s] = ld4(Q + (size_t)rows * a.d + dim);
      gr[s] = ld4(dO + (size_t)rows * a.d + dim);
    }
    float qt[4][DT], gt[4][DT];
    f4 inf[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = __shfl(rows, 4 * quad + i);
      inf[i] = info[r];
      ld_chunk<DT>(Q + (size_t)r * a.d + c, qt[i]);
      ld_chunk<DT>(dO + (size_t)r * a.d + c, gt[i]);
    }
    tq += dt_;
    hd += dh;
    if (hd >= a.hs) { hd -= a.hs; ++tq; }
    ql = q0 + tq;
    if (e0 + 16 * NW_KEY < ne) th = row_of(min(ql, q1 - 1));
    const f4 s = dot16<DT>(qr, k), dp = dot16<DT>(gr, v);  // rows: query rows 4*quad + i, column: key n
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int qi = __shfl(qls, 4 * quad + i);
      const bool on = qi < q1 && qi >= qlo && qi < qhi;
      const float p = on ? __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], a.sl2, -inf[i][0])) : 0.f;
      const float ds = p * (inf[i][2] * dp[i] - inf[i][1]) * a.scale, pw = p * inf[i][2];
#pragma unroll
      for (int b = 0; b < DT; ++b) {
        dv[b] = mfma4(gt[i][b], pw, dv[b]);
        dk[b] = mfma4(qt[i][b], ds, dk[b]);
      }
    }
  }
  if (__builtin_expect(!__all(finite_sums<DT>(dk) && finite_sums<DT>(dv)), 0)) {  // once more, one query row at a time
#pragma unroll
    for (int b = 0; b < DT; ++b) dk[b] = dv[b] = f4{0.f, 0.f, 0.f, 0.f};
    const int thr = thread_again(), n = thr & 15, quad = thr >> 4 & 3, c = n * DT < a.d ? n * DT : 0;
#pragma unroll 1
    for (int e0 = 16 * wid; e0 < ne; e0 += 16 * NW_KEY) {
      const int e = min(e0 + n, ne - 1), t = q0 + e / a.hs, qls = e0 + n < ne ? t : q1;
      const int row = (list ? list[t] : a.bv.perm[t]) * a.Hq + g * a.hs + e % a.hs;
      f4 x[DT], pw, ds;
      ld_row<T, DT>(Q + (size_t)row * a.d, a.d, true, x, quad);
      const f4 s = dot16<DT>(x, k);
      ld_row<T, DT>(dO + (size_t)row * a.d, a.d, true, x, quad);
      const f4 dp = dot16<DT>(x, v);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f4 inf = info[__shfl(row, 4 * quad + i)];
        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], a.sl2, -inf[0]));
        ds[i] = p * (inf[2] * dp[i] - inf[1]) * a.scale;
        pw[i] = p * inf[2];
      }
#pragma unroll 1
      for (int r = 0; r < 16; ++r) {
        const int qi = __shfl(qls, r);
        const bool mine = qi < q1 && qi >= qlo && qi < qhi;
        const size_t off = (size_t)__shfl(row, r) * a.d + c;
        add_alone<DT>(dv, dO + off, of_row(pw, r), mine);
        add_alone<DT>(dk, Q + off, of_row(ds, r), mine);
      }
    }
  }
  // sums of the wavefronts in a fixed tree: the upper half hands its sums to the lower half, and so on
  for (int h = NW_KEY / 2; h >= 1; h /= 2) {
    if (wid >= h && wid < 2 * h) {
      acc_put<DT>(part[wid - h][0][n], dk);
      acc_put<DT>(part[wid - h][1][n], dv);
    }
    __syncthreads();
    if (wid < h) {
      acc_add<DT>(part[wid][0][n], dk);
      acc_add<DT>(part[wid][1][n], dv);
    }
    __syncthreads();
  }
  if (wid != 0 || !key_on) return;
  acc_put<DT>(oK + (size_t)n * ostride, dk, a.d);
  acc_put<DT>(oV + (size_t)n * ostride, dv, a.d);
}

// dK[tok] = window part + the selection chunks in order + (the compression splits in order) / count (gradient of the mean
// pool), scattered back to caller order.  One thread per (sorted position, 4 elements of the row).
struct FinishArgs {
  BlkView bv;
  int Hkv, d, splits;
  const int32_t *chunk_start, *part_row_start;
  const float *dKs, *dVs, *pK, *pV, *dKc, *dVc;
  void *dK, *dV;
};
template <typename T>
__global__ __launch_bounds__(256) void g_bwd_finish(FinishArgs a) {
  const int row = a.Hkv * a.d, per = row / 4;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (size_t)a.bv.N * per) return;
  const int pos = (int)(i / per), f = (int)(i % per) * 4, g = f / a.d, dim = f % a.d;
  f4 k = ld4(a.dKs + (size_t)pos * row + f), v = ld4(a.dVs + (size_t)pos * row + f);
  const int b = a.bv.tok_slc[pos], key = g * a.bv.Ns + b, klen = a.bv.slc_start[b + 1] - a.bv.slc_start[b];
  const int nch = a.chunk_start[key + 1] - a.chunk_start[key];
  const size_t r0 = (size_t)a.part_row_start[key] + (pos - a.bv.slc_start[b]);
#pragma unroll 4
  for (int c = 0; c < nch; ++c) {
    const size_t off = (r0 + (size_t)c * klen) * a.d + dim;
    k += ld4(a.pK + off);
    v += ld4(a.pV + off);
  }
  const int cb = a.bv.tok_cmp[pos];
  const float inv = 1.0f / (float)(a.bv.cmp_start[cb + 1] - a.bv.cmp_start[cb]);
  f4 ck = {0.f, 0.f, 0.f, 0.f}, cv = ck;
#pragma unroll 4
  for (int s = 0; s < a.splits; ++s) {
    const size_t off = ((size_t)s * a.bv.Nc + cb) * row + f;
    ck += ld4(a.dKc + off);
    cv += ld4(a.dVc + off);
  }
  const size_t dst = (size_t)a.bv.perm[pos] * row + f;
  st4((T *)a.dK + dst, k + ck * inv);
  st4((T *)a.dV + dst, v + cv * inv);
}

struct GenericPlan {
  size_t ks, vs, kc, vc, ob, lse, idx, info, dks, dvs, pk, pv, dkc, dvc, sel, total;
  int chunk_len, max_chunks, splits;
};

GenericPlan plan(const ssa_ctx &c, bool bwd) {
  GenericPlan p{};
  const ssa_blocks *b = c.blk;
  const size_t esz = c.dtype == SSA_F32 ? 4 : 2;
  const size_t kv = align_up((size_t)c.N * c.Hkv * c.d * 4 + 4, 256);
  const size_t kvc = align_up((size_t)b->Nc * c.Hkv * c.d * 4 + 4, 256);
  size_t off = 0;
  auto take = [&](size_t n) { size_t r = off; off += align_up(n, 256); return r; };
  p.ks = take(kv); p.vs = take(kv); p.kc = take(kvc); p.vc = take(kvc);
  if (!bwd) {
    p.ob = take((size_t)3 * c.N * c.Hq * c.d * esz + 4);
    p.lse = take((size_t)3 * c.N * c.Hq * 4 + 4);
    p.idx = take((size_t)c.N * c.Hkv * c.T * 4 + 4);
  } else {
    p.info = take((size_t)3 * c.N * c.Hq * 16);
    p.dks = take(kv); p.dvs = take(kv);
    // selection lists are cut into chunks whose partial dK, dV are added in order; chunks grow until the partial sums fit in
    // about 1 GiB (rows <= slc_tok_max * full chunks + one partly filled chunk per key)
    const size_t entries = (size_t)c.N * c.Hkv * c.T, keys = (size_t)c.Hkv * b->Ns;
    size_t rows;
    for (p.chunk_len = 256;; p.chunk_len *= 2) {
      rows = (size_t)b->slc_tok_max * (entries / p.chunk_len + 1) + (size_t)c.N * c.Hkv;
      if (rows * c.d * 8 <= ((size_t)1 << 30) || p.chunk_len >= (1 << 20)) break;
    }
    p.max_chunks = (int)(entries / p.chunk_len + keys + 1);
    p.pk = take(rows * c.d * 4); p.pv = take(rows * c.d * 4);
    // compression branch: the query range in parts, so that about 512 workgroups share it, of 128 query rows or more
    const long long wgs = (long long)((b->Nc + 15) / 16) * c.Hkv, most = (long long)c.N * c.hs / 128 + 1;
    long long sp = (512 + wgs - 1) / (wgs > 0 ? wgs : 1);
    sp = sp > most ? most : sp;
    p.splits = (int)(sp < 1 ? 1 : sp > 64 ? 64 : sp);
    p.dkc = take(kvc * p.splits); p.dvc = take(kvc * p.splits);
    p.sel = take(sel_index_bytes(c.N, c.Hkv, c.T, b->Ns));
  }
  p.total = off;
  return p;
}

// Tokens per workgroup of the score kernel: a tile's worth, fewer where their score rows would not fit the LDS.
int score_tokens(const ssa_ctx &c) {
  int tw = tokens_per_tile(c.hs);
  while (tw > 1 && score_lds_bytes(tw, c.blk->s_max) > 64 * 1024) tw /= 2;
  return tw;
}

template <typename T, int DT>
int forward_t(const ssa_ctx &c, const void *q, const void *k, const void *v, const void *gates, void *out, float *lse,
              int32_t *topk_idx, void *out_branch, char *ws) {
  const GenericPlan p = plan(c, false);
  const BlkView bv = view_of(c.blk);
  float *Ks = (float *)(ws + p.ks), *Vs = (float *)(ws + p.vs), *Kc = (float *)(ws + p.kc), *Vc = (float *)(ws + p.vc);
  void *Ob = out_branch ? out_branch : (void *)(ws + p.ob);
  float *L = lse ? lse : (float *)(ws + p.lse);
  int32_t *I = topk_idx ? topk_idx : (int32_t *)(ws + p.idx);
  const int tw = score_tokens(c), tpt = tokens_per_tile(c.hs);
  const size_t lds = score_lds_bytes(tw, c.blk->s_max);
  if (lds > 150 * 1024) return SSA_ERR_UNSUPPORTED;
  static std::once_flag once;
  std::call_once(once, [] {
    (void)hipFuncSetAttribute((const void *)g_scores_topk<T, DT>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  });
  const float sl2 = c.scale * LOG2E_F;
  const dim3 grid((unsigned)((c.N + tpt - 1) / tpt * tiles_per_token(c.hs)), c.Hkv);
  g_sort_pool<T><<<c.blk->Nc, 256, 0, c.stream>>>((const T *)k, (const T *)v, bv, c.Hkv * c.d, Ks, Vs, Kc, Vc, nullptr);
  FwdArgs a{q, gates, bv, I, c.Hq, c.Hkv, c.hs, c.d, c.T, sl2, Kc, Vc, Ob, out, L};
  g_cmp_fwd<T, DT><<<grid, 64 * NW, 0, c.stream>>>(a);
  ScoreArgs sa{q, bv, Kc, L, I, c.Hq, c.Hkv, c.hs, c.d, c.T, tw, c.blk->s_max, sl2};
  g_scores_topk<T, DT><<<dim3((c.N + tw - 1) / tw, c.Hkv), 64 * NW, lds, c.stream>>>(sa);
  a.K = Ks; a.V = Vs;
  g_slc_win_fwd<T, DT><<<grid, 64 * NW, union_lds_bytes(tpt, c.T), c.stream>>>(a);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}

template <typename T, int DT>
int backward_t(const ssa_ctx &c, const void *q, const void *k, const void *v, const void *gates, const void *out_branch,
               const float *lse, const int32_t *topk_idx, const void *dout, void *dq, void *dk, void *dv, void *dgates,
               char *ws) {
  const GenericPlan p = plan(c, true);
  const BlkView bv = view_of(c.blk);
  float *Ks = (float *)(ws + p.ks), *Vs = (float *)(ws + p.vs), *Kc = (float *)(ws + p.kc), *Vc = (float *)(ws + p.vc);
  f4 *info = (f4 *)(ws + p.info);
  float *dKs = (float *)(ws + p.dks), *dVs = (float *)(ws + p.dvs), *dKc = (float *)(ws + p.dkc), *dVc = (float *)(ws + p.dvc);
  float *pK = (float *)(ws + p.pk), *pV = (float *)(ws + p.pv);
  const int tpt = tokens_per_tile(c.hs), row = c.Hkv * c.d;
  const float sl2 = c.scale * LOG2E_F;
  const dim3 grid((unsigned)((c.N + tpt - 1) / tpt * tiles_per_token(c.hs)), c.Hkv);
  const SelIndex sel = sel_index_carve(ws + p.sel, c.N, c.Hkv, c.T, c.blk->Ns, p.chunk_len, BC_CHUNK);
  g_sort_pool<T><<<c.blk->Nc, 256, 0, c.stream>>>((const T *)k, (const T *)v, bv, row, Ks, Vs, Kc, Vc, sel.ticket);
  DqArgs a{q, dout, out_branch, gates, bv, topk_idx, c.Hq, c.Hkv, c.hs, c.d, c.T, c.scale, sl2, Ks, Vs, Kc, Vc, lse, dq, dgates, info};
  g_bwd_dq<T, DT><<<grid, 64 * NW, union_lds_bytes(tpt, c.T), c.stream>>>(a);
  const int rc = sel_index_build(topk_idx, c.blk->perm, c.blk->slc_start, c.N, c.Hkv, c.T, c.blk->Ns, sel, true, false, true, false, c.stream);
  if (rc != SSA_OK) return rc;
  DkvArgs b{q, dout, bv, c.Hq, c.Hkv, c.hs, c.d, c.scale, sl2, Ks, Vs, Kc, Vc, info, sel.list, sel.chunk_start,
            sel.part_row_start, sel.order, (c.blk->slc_tok_max + 15) / 16, p.splits, 0, 0, 0, dKs, dVs, pK, pV, dKc, dVc};
  b.n_win = (long long)((c.N + 15) / 16) * c.Hkv;
  b.n_slc = (long long)p.max_chunks * b.slc_tiles;
  const long long wgs = b.n_win + b.n_slc + (long long)((c.blk->Nc + 15) / 16) * c.Hkv * p.splits;
  // a selection chunk has workgroups for the longest block's tiles: one long block among many short ones makes more of them than
  // one launch can have (2^32 threads)
  constexpr long long MOST = (1ll << 31) / (64 * nw_key<DT>());
  for (; b.first < wgs; b.first += MOST)
    g_bwd_dkv<T, DT><<<(unsigned)(wgs - b.first < MOST ? wgs - b.first : MOST), 64 * nw_key<DT>(), 0, c.stream>>>(b);
  FinishArgs f{bv, c.Hkv, c.d, p.splits, sel.chunk_start, sel.part_row_start, dKs, dVs, pK, pV, dKc, dVc, dk, dv};
  const size_t items = (size_t)c.N * row / 4;
  g_bwd_finish<T><<<(unsigned)((items + 255) / 256), 256, 0, c.stream>>>(f);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}

// blocks of 16 dims a row is padded to in the registers
#define SSA_GENERIC_DISPATCH(fn, ...)                                                                  \
  (c.dtype == SSA_F32                                                                                  \
       ? (c.d <= 16 ? fn<float, 1>(__VA_ARGS__) : c.d <= 32 ? fn<float, 2>(__VA_ARGS__)                \
          : c.d <= 64 ? fn<float, 4>(__VA_ARGS__) : fn<float, 8>(__VA_ARGS__))                         \
       : (c.d <= 16 ? fn<uint16_t, 1>(__VA_ARGS__) : c.d <= 32 ? fn<uint16_t, 2>(__VA_ARGS__)          \
          : c.d <= 64 ? fn<uint16_t, 4>(__VA_ARGS__) : fn<uint16_t, 8>(__VA_ARGS__)))

}  // namespace

size_t generic_forward_workspace(const ssa_ctx &c) { return plan(c, false).total; }
size_t generic_backward_workspace(const ssa_ctx &c) { return plan(c, true).total; }

int generic_forward(const ssa_ctx &c, const void *q, const void *k, const void *v, const void *gates, void *out,
                    float *lse, int32_t *topk_idx, void *out_branch, void *ws, size_t ws_bytes) {
  if (ws_bytes < plan(c, false).total) return SSA_ERR_WORKSPACE;
  if (c.N == 0) return SSA_OK;
  ProfScope ps(PROF_GENERIC, c.stream);
  return SSA_GENERIC_DISPATCH(forward_t, c, q, k, v, gates, out, lse, topk_idx, out_branch, (char *)ws);
}

int generic_backward(const ssa_ctx &c, const void *q, const void *k, const void *v, const void *gates,
                     const void *out_branch, const float *lse, const int32_t *topk_idx, const void *dout, void *dq,
                     void *dk, void *dv, void *dgates, void *ws, size_t ws_bytes) {
  if (ws_bytes < plan(c, true).total) return SSA_ERR_WORKSPACE;
  if (c.N == 0) return SSA_OK;
  ProfScope ps(PROF_GENERIC, c.stream);
  return SSA_GENERIC_DISPATCH(backward_t, c, q, k, v, gates, out_branch, lse, topk_idx, dout, dq, dk, dv, dgates, (char *)ws);
}

int launch_topk_from_scores(const ssa_ctx &c, const float *scores, int32_t *topk_idx) {
  if (c.N == 0) return SSA_OK;
  const int s_max = c.blk->s_max;
  const size_t lds = ((size_t)s_max + ((size_t)s_max + 31) / 32 + 4) * 4;
  if (lds > 60000) return SSA_ERR_UNSUPPORTED;
  g_topk_from_scores<<<c.N * c.Hkv, WAVE, lds, c.stream>>>(scores, view_of(c.blk), c.Hkv, c.T, s_max, c.blk->inv_perm,
                                                          topk_idx);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}
