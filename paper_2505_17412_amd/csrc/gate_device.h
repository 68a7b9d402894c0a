// Device code of the gate predictor's forward pass by workgroups that split the contraction (gate.hip): a kernel of its own, or workgroups
// beside those of the projections of the same rows (linear.hip).
#pragma once

#include "mfma_common.h"
#include "mfma_qc.h"

constexpr int JP = 64;  // padded gate count (columns of dz and of the padded weights)

struct GateJob {
  const bf16_t *x, *w, *bias;  // [N][Dm], [Dm][J], [J]
  int N, Dm, J;
  bf16_t *gates;               // [N][J]
  int first;                   // beside another kernel: its first workgroup for the gates
  __host__ __device__ int blocks() const { return (J + 15) / 16; }
};

// The lane's bias of column block nb, for before the first store: behind one the load waits for it.
__device__ inline float gate_bias(const GateJob &a, int nb) { return bf16_to_f32(a.bias[min(16 * nb + (int)(threadIdx.x & 15), a.J - 1)]); }
// gates[tok][j] = sigmoid(z + b); C layout: lane holds gate column 16*nb + n of tokens t0 + 4*quad + i
__device__ inline void gate_store(const GateJob &a, int t0, int nb, const f32x4 &z, float b) {
  const int n = threadIdx.x & 15, quad = threadIdx.x >> 4 & 3, j = 16 * nb + n;
  if (j >= a.J) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int t = t0 + 4 * quad + i;
    if (t < a.N) a.gates[(size_t)t * a.J + j] = f32_to_bf16(1.0f / (1.0f + __expf(-(z[i] + b))));
  }
}

// Workgroup wg of the split form: 256 threads (or as many of a larger one, with LDS of their own); each of the four wavefronts takes a quarter of the contraction of the same 32 tokens, added
// in order through LDS.  WT: wt holds the weights as [16*NB][Dm] (transposed), or they are read as they are, for J a multiple of 8: 32 rows
// at a time go through the wavefront's own LDS and come back as transposed operands.
template <int NB> constexpr size_t gate_part_bytes() { return (size_t)4 * 2 * NB * 64 * sizeof(f32x4); }
template <int NB, bool WT> constexpr size_t gate_split_lds() { return gate_part_bytes<NB>() + (WT ? 0 : (size_t)4 * 2 * TileGeom<JP>::ROW_ELEMS * 2); }

template <int NB, bool WT>
__device__ __forceinline__ void gate_split_tile(const GateJob &a, const bf16_t *wt, int wg, unsigned char *lds) {
  using G = TileGeom<JP>;
  f32x4 *part = (f32x4 *)lds;  // [4][2 * NB][64]
  const int wid = threadIdx.x >> 6 & 3, lane = threadIdx.x & 63, n = lane & 15, quad = lane >> 4;
  bf16_t *tiles = (bf16_t *)(lds + gate_part_bytes<NB>()) + wid * 2 * G::ROW_ELEMS;
  const int t0 = wg * 32, Dm = a.Dm, J = a.J;
  const bf16_t *xr[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) xr[h] = a.x + (size_t)min(t0 + 16 * h + n, a.N - 1) * Dm + 8 * quad;  // rows past the end
  f32x4 acc[2][NB];                                                                         // repeat the last token
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[h][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int trips = Dm / 128;  // d_model is a multiple of 128: four contraction steps per trip
  const int k_begin = trips * wid / 4, k_end = trips * (wid + 1) / 4;
  constexpr int IW = NB;       // 16-byte pieces of 32 weight rows per lane: 4 * J of them, J <= 16 * NB
  int piece[IW], slot[IW];     // a lane's pieces in memory, and where they go (past the last: the last again)
  if constexpr (!WT) {
#pragma unroll
    for (int i = 0; i < IW; ++i) {
      piece[i] = 8 * min(lane + 64 * i, 4 * J - 1);
      slot[i] = G::row_off(piece[i] / J, piece[i] % J / 8);
    }
  }
  for (int k4 = k_begin; k4 < k_end; ++k4) {
    bf16x8 av[2][4], wv[4][IW];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      av[0][u] = ld8(xr[0] + 128 * k4 + 32 * u);
      av[1][u] = ld8(xr[1] + 128 * k4 + 32 * u);
      if constexpr (!WT)
#pragma unroll
        for (int i = 0; i < IW; ++i) wv[u][i] = ld8(a.w + (size_t)(128 * k4 + 32 * u) * J + piece[i]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      bf16_t *tile = tiles + (u & 1) * G::ROW_ELEMS;
      if constexpr (!WT)
#pragma unroll
        for (int i = 0; i < IW; ++i) *reinterpret_cast<bf16x8 *>(tile + slot[i]) = wv[u][i];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        bf16x8 bv;
        if constexpr (WT) bv = ld8(wt + (size_t)(16 * nb + n) * Dm + 128 * k4 + 32 * u + 8 * quad);
        else bv = lds_tr_operand<JP>(tile, nb);  // (columns from J on: whatever lies there, for nobody)
        acc[0][nb] = mfma16(av[0][u], bv, acc[0][nb]);
        acc[1][nb] = mfma16(av[1][u], bv, acc[1][nb]);
      }
    }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) part[(wid * 2 * NB + h * NB + nb) * 64 + lane] = acc[h][nb];
  __syncthreads();
  for (int it = wid; it < 2 * NB; it += 4) {  // the wavefronts take the tiles in turn
    f32x4 p[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) p[w] = part[(w * 2 * NB + it) * 64 + lane];
    gate_store(a, t0 + 16 * (it / NB), it % NB, ((p[0] + p[1]) + p[2]) + p[3], gate_bias(a, it % NB));
  }
}

// The gates as workgroups beside a projection's (gate.hip): whether that form takes them, checked as by ssa_gate_forward.
bool gate_beside(const ssa_params_t *p, int d_model, const void *x, const void *w, const void *bias, void *gates, GateJob *out);
