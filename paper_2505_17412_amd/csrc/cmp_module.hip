// Learned sparse 3D compression module for gfx950: x + PE, sparse 3x3x3 convolution, mean pool (paper, Sec. "Sparse 3D
// Compression", eq. (5)), forward and backward.
//
// Readings (the paper gives the three operations and nothing else): PE is a table [m_cmp^3][C] indexed by the
// token's place inside its compression block, row ((x mod m)*m + (y mod m))*m + (z mod m); the convolution is a
// submanifold 3x3x3 one over the sparse volume of the token's batch item (outputs at active sites, inactive
// neighbours contribute nothing), C -> C channels with bias, C = H_kv * head_dim; w[o] is [C_in][C_out] for
// offset o = ((dx+1)*3 + (dy+1))*3 + (dz+1) and multiplies the token at coords + (dx,dy,dz); the mean runs over
// the active tokens of the compression block.  Coordinates must be distinct inside an item.
//
// Layout: everything is done in the sorted (Morton) token order of the block structure.  The neighbour of a
// token is found by binary search of its Morton key among the sorted keys the handle keeps.  The convolution is a
// gather-GEMM on the matrix cores: a wavefront owns 64 tokens (four 16-row MFMA tiles) and 32 output channels,
// and for each of the 27 offsets multiplies the gathered neighbour rows (A operand, 16 bytes per lane straight
// from memory) with the offset's C x C weights (B operand, contraction index contiguous).  The data gradient is
// the same kernel on mirrored offsets with the weights read the other way round; the weight gradient contracts
// over tokens, its two operands come from row-major LDS tiles through the transposing LDS read.  No floating
// point atomics anywhere: partial sums are written per chunk and added in a fixed order.
//
// A layer runs the module on its keys and on its values: every launch takes one or two tensors (blockIdx.z), which
// share the neighbour table and together fill the chip where one alone does not.
#include "mfma_common.h"
#include "mfma_qc.h"
#include "profile.h"
#include "cmp_internal.h"

namespace {

// one entry per tensor of a launch; blockIdx.z picks it
template <class T> struct Pair { T v[2]; };

__device__ inline uint32_t compact3(uint64_t v64) {  // bits 0,3,6,.. of v -> bits 0,1,2,..
  uint32_t v = (uint32_t)v64 & 0x09249249u;
  v = (v | (v >> 2)) & 0x030C30C3u;
  v = (v | (v >> 4)) & 0x0300F00Fu;
  v = (v | (v >> 8)) & 0x030000FFu;
  v = (v | (v >> 16)) & 0x3FFu;
  return v;
}
__device__ inline uint32_t spread3m(uint32_t v) {
  v &= 0x3FFu;
  v = (v | (v << 16)) & 0x030000FFu;
  v = (v | (v << 8)) & 0x0300F00Fu;
  v = (v | (v << 4)) & 0x030C30C3u;
  v = (v | (v << 2)) & 0x09249249u;
  return v;
}
struct Site { int item, x, y, z; };
__device__ inline Site decode(uint64_t key, int bits) {
  const uint64_t code = key & ((1ull << (3 * bits)) - 1ull);
  return Site{(int)(key >> (3 * bits)), (int)compact3(code >> 2), (int)compact3(code >> 1), (int)compact3(code)};
}

// What a pass needs before its convolution, in one launch: the neighbour table, U of the tensors, and in the forward pass the transposed weights
// (10.7k tokens: in three launches 18.8 us, 11.7 in one).  Workgroups of 256 items each, one kind after the other.
struct PrepareArgs {
  const uint64_t *keys;
  const int32_t *item_start, *perm;
  int N, G, bits, C, m;
  int32_t *nbr;
  Pair<const bf16_t *> x, pe, w;
  Pair<bf16_t *> U, wt;
  unsigned nbr_wgs, pe_wgs, wt_wgs;  // of the table; per tensor of the others
};

// nbr[pos][o] = sorted position of the token at coords(pos) + offset o in the same item, or -1.  One thread per
// (pos, o): a binary search of the neighbour's key inside the item's range of the sorted keys.
__device__ inline void find_neighbor(const PrepareArgs &a, size_t i) {
  if (i >= (size_t)a.N * 27) return;
  const uint64_t *__restrict__ keys = a.keys;
  const int bits = a.bits, pos = (int)(i / 27), o = (int)(i % 27);
  const Site s = decode(keys[pos], bits);
  const int x = s.x + o / 9 - 1, y = s.y + o / 3 % 3 - 1, z = s.z + o % 3 - 1;
  int found = -1;
  if ((unsigned)x < (unsigned)a.G && (unsigned)y < (unsigned)a.G && (unsigned)z < (unsigned)a.G) {
    const uint64_t want = ((uint64_t)s.item << (3 * bits)) |
                          (uint64_t)((spread3m((uint32_t)x) << 2) | (spread3m((uint32_t)y) << 1) | spread3m((uint32_t)z));
    int lo = a.item_start[s.item];
    const int e = a.item_start[s.item + 1];
    int hi = e;  // first position in [lo, e) whose key is >= want
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (keys[mid] < want) lo = mid + 1; else hi = mid;
    }
    if (lo < e && keys[lo] == want) found = lo;
  }
  a.nbr[i] = found;
}

// U[pos] = x[perm[pos]] + PE[place of the token inside its block]   (bf16, sorted order)
__device__ inline void add_pe(const PrepareArgs &a, int tensor, size_t i) {
  const bf16_t *__restrict__ x = a.x.v[tensor], *__restrict__ pe = a.pe.v[tensor];
  const int per = a.C / 8, m = a.m;
  if (i >= (size_t)a.N * per) return;
  const int pos = (int)(i / per), c0 = (int)(i % per) * 8;
  const Site s = decode(a.keys[pos], a.bits);
  const int p = ((s.x & (m - 1)) * m + (s.y & (m - 1))) * m + (s.z & (m - 1));
  const bf16x8 u = ld8(x + (size_t)a.perm[pos] * a.C + c0), v = ld8(pe + (size_t)p * a.C + c0);
  bf16x8 r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r[j] = (__bf16)((float)u[j] + (float)v[j]);
  *reinterpret_cast<bf16x8 *>(a.U.v[tensor] + (size_t)pos * a.C + c0) = r;
}

__global__ __launch_bounds__(256) void c_prepare(PrepareArgs a) {
  unsigned wg = blockIdx.x;
  if (wg < a.nbr_wgs) return find_neighbor(a, (size_t)wg * 256 + threadIdx.x);
  wg -= a.nbr_wgs;
  if (a.wt_wgs == 0) return add_pe(a, wg / a.pe_wgs, (size_t)(wg % a.pe_wgs) * 256 + threadIdx.x);
  const int tensor = wg / (a.pe_wgs + a.wt_wgs);
  wg %= a.pe_wgs + a.wt_wgs;
  if (wg < a.pe_wgs) return add_pe(a, tensor, (size_t)wg * 256 + threadIdx.x);
  // wt[o][c_out][c_in] = w[o][c_in][c_out]
  const int C = a.C;
  const size_t i = (size_t)(wg - a.pe_wgs) * 256 + threadIdx.x;
  if (i >= (size_t)27 * C * C) return;
  const int ci = (int)(i % C), co = (int)(i / C % C), o = (int)(i / ((size_t)C * C));
  a.wt.v[tensor][i] = a.w.v[tensor][((size_t)o * C + ci) * C + co];
}

// Gather-GEMM: out[pos][n] = bias[n] + sum_o sum_k in[nbr[pos][o']][k] * Bw[o][n][k], o' = o (forward) or 26 - o
// (data gradient: the token that took `pos` as its neighbour o sits at the mirrored offset).  Bw holds, per offset,
// a [C][C] matrix with the contraction index contiguous.
struct ConvSrc { const bf16_t *in, *w, *bias; float *out; };
template <int C, bool MIRROR, int MT, int NBW>
__global__ __launch_bounds__(256) void c_conv(Pair<ConvSrc> srcs, const int32_t *__restrict__ nbr, int N) {
  const ConvSrc cs = srcs.v[blockIdx.z];
  const bf16_t *__restrict__ in = cs.in, *__restrict__ Bw = cs.w, *__restrict__ bias = cs.bias;
  float *__restrict__ out = cs.out;
  const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, quad = lane >> 4;
  const int pos0 = (blockIdx.x * 4 + wid) * 16 * MT;  // a wavefront owns MT tiles of 16 tokens: every weight operand
  if (pos0 >= N) return;                               // it loads feeds MT matrix instructions
  const int nb0 = blockIdx.y * NBW;                    // blockIdx.y: which NBW blocks of 16 output channels
  f32x4 acc[MT][NBW];
#pragma unroll
  for (int a = 0; a < MT; ++a)
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) acc[a][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  int tok[MT], nxt[MT];
#pragma unroll
  for (int a = 0; a < MT; ++a) {
    tok[a] = pos0 + 16 * a + n;
    nxt[a] = tok[a] < N ? nbr[(size_t)tok[a] * 27 + (MIRROR ? 26 : 0)] : -1;
  }
  for (int o = 0; o < 27; ++o) {
    // the neighbour indices of the next offset are requested before this offset's rows are used: the two dependent
    // loads (index, then row) of consecutive offsets overlap
    int src[MT];
    bool some = false;
#pragma unroll
    for (int a = 0; a < MT; ++a) {
      src[a] = nxt[a];
      some = some || src[a] >= 0;
      if (o + 1 < 27) nxt[a] = tok[a] < N ? nbr[(size_t)tok[a] * 27 + (MIRROR ? 25 - o : o + 1)] : -1;
    }
    if (!__any(some)) continue;
    const bf16_t *Bo = Bw + (size_t)o * C * C;
#pragma unroll
    for (int ks = 0; ks < C / 32; ++ks) {
      bf16x8 av[MT];
#pragma unroll
      for (int a = 0; a < MT; ++a) av[a] = src[a] >= 0 ? ld8(in + (size_t)src[a] * C + 32 * ks + 8 * quad) : zero8();
#pragma unroll
      for (int nb = 0; nb < NBW; ++nb) {
        const bf16x8 bv = ld8(Bo + (size_t)(16 * (nb0 + nb) + n) * C + 32 * ks + 8 * quad);
#pragma unroll
        for (int a = 0; a < MT; ++a) acc[a][nb] = mfma16(av[a], bv, acc[a][nb]);
      }
    }
  }
  // C layout: lane holds output channel 16*(nb0 + nb) + n of tokens pos0 + 16*a + 4*quad + i
#pragma unroll
  for (int nb = 0; nb < NBW; ++nb) {
    const int ch = 16 * (nb0 + nb) + n;
    const float bs = bias ? bf16_to_f32(bias[ch]) : 0.f;
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = pos0 + 16 * a + 4 * quad + i;
        if (t < N) out[(size_t)t * C + ch] = acc[a][nb][i] + bs;
      }
  }
}

// The same gather-GEMM for C = 128: a workgroup owns TOK tokens, wavefront w the output channels 32w .. 32w+31.  Per offset
// the TOK gathered rows go through LDS (two buffers, one barrier per offset) and are read by all four wavefronts as
// conflict-free row operands; the weights of a wavefront's channels are nobody else's, so they go from memory straight into
// its operand registers.  Rows and weights of the next offset are in flight during the products of this one, the row indices
// taken from a copy of the tile's neighbour table in LDS.  Row r of a 16-row MFMA tile stands for LDS row
// 8*(r >> 2) + 4*a + (r & 3) of its 32-row tile (a = which half), for tokens and for channels alike; the store at the end
// undoes that numbering.
// Bound: the chain index -> gathered row -> LDS -> product of an offset, with one or two wavefronts per SIMD to cover it; about half
// of the gathered rows of a surface are zeros.  At 64 tokens the products of an offset are too short to hide a weight loaded behind
// its last use, so the next offset's weights have registers of their own, and rows are requested two offsets ahead.  At 128 tokens
// those registers would cost the second wavefront, so a weight is loaded again in place and rows are one offset ahead.
// Convolution forward of keys and values, rows one -> two ahead: 7 k tokens (64 per workgroup) 91 -> 72 us; 128 per workgroup
// 10.7 k 123 -> 115, but 17 k 136 -> 147, 30 k 155 -> 170, 60 k 312 -> 331.  With loads under conditions and one ahead: 7 k 88,
// 10.7 k 121, 17 k 137, 30 k 162, 60 k 322.  Eight wavefronts that share 128 tokens by halves fetch the weights twice: 140 at
// 10.7 k, 480 at 60 k.
template <bool MIRROR, int TOK>
__global__ __launch_bounds__(256) void c_conv128(Pair<ConvSrc> srcs, const int32_t *__restrict__ nbr, int N, size_t part_stride) {
  constexpr int C = 128, MT = TOK / 16, AI = TOK / 16;  // AI: gathered 16-byte items per thread (TOK x 16 / 256)
  using G = TileGeom<C>;
  const ConvSrc cs = srcs.v[blockIdx.z];
  const bf16_t *__restrict__ in = cs.in, *__restrict__ Bw = cs.w;
  __shared__ __align__(16) bf16_t sa[2][(TOK / 32) * G::ROW_ELEMS];
  __shared__ int any_flag[27];
  __shared__ int32_t snbr[TOK * 27];
  const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, quad = lane >> 4;
  const int pos0 = blockIdx.x * TOK;
  // which offsets have a neighbour for any of the tokens (workgroup-uniform skip)
  if (threadIdx.x < 27) any_flag[threadIdx.x] = 0;
  __syncthreads();
  for (int i = threadIdx.x; i < TOK * 27; i += 256) {
    const int t = pos0 + i / 27, o = i % 27;
    const int32_t v = t < N ? nbr[(size_t)t * 27 + o] : -1;
    snbr[i] = v;
    if (v >= 0) any_flag[MIRROR ? 26 - o : o] = 1;
  }
  __syncthreads();
  uint32_t used = (uint32_t)__ballot(lane < 27 && any_flag[lane < 27 ? lane : 0] != 0);
  if (gridDim.y > 1) {  // this workgroup's share of them
    const int total = __popc(used), first = total * (int)blockIdx.y / (int)gridDim.y, end = total * (int)(blockIdx.y + 1) / (int)gridDim.y;
    uint32_t later = used;
    for (int i = 0; i < end; ++i) {
      if (i < first) used &= used - 1u;
      later &= later - 1u;
    }
    used ^= later;
  }
  f32x4 acc[MT][2];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) acc[mt][0] = acc[mt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  // weights of one offset; with 64 tokens those of the next one have registers of their own, and so have the rows of another offset
  constexpr bool AHEAD = TOK == 64;
  struct Weights { bf16x8 v[2][C / 32]; };
  Weights wa, wb;
  struct Rows { bf16x8 v[AI]; uint32_t missing; };
  Rows ra, rb;
  const int wrow = 32 * wid + 8 * (n >> 2) + (n & 3);  // channel of half 0; half 1 is 4 further
  const bf16_t *Bl = Bw + (size_t)wrow * C + 8 * quad;
  auto fetch_weights = [&](int o, int ks, Weights &w) {
#pragma unroll
    for (int a = 0; a < 2; ++a) w.v[a][ks] = ld8(Bl + (size_t)o * C * C + 4 * a * C + 32 * ks);
  };
  // (loads are unconditional, a missing neighbour's from row 0 and an offset past the last from offset 26: behind a branch the
  // compiler cannot count what is outstanding, and the products would wait for the rows just requested)
  auto fetch_rows = [&](int o_, Rows &r) {
    const int o = min(o_, 26), oo = MIRROR ? 26 - o : o;
    r.missing = 0u;
#pragma unroll
    for (int i = 0; i < AI; ++i) {
      const int it = threadIdx.x + 256 * i;
      const int src = snbr[(it / 16) * 27 + oo];
      r.missing |= src < 0 ? 1u << i : 0u;
      r.v[i] = ld8(in + (uint32_t)(max(src, 0) * C + 8 * (it % 16)));
    }
  };
  auto next = [&](int o) {  // the next offset in use, 27 behind the last
    const uint32_t later = used & ~((2u << o) - 1u);
    return later ? __builtin_ctz(later) : 27;
  };
  // one offset: its rows (in registers) to LDS buffer `buf`, the rows of the next offset (AHEAD: the one after it) requested in their
  // place, the next offset's weights requested, the products; with cur and nxt the same registers a weight is loaded again as soon as
  // this offset is done with it
  int o = used ? __builtin_ctz(used) : 27, o1 = next(min(o, 27));
  auto step = [&](int buf, Weights &cur, Weights &nxt, Rows &r) {
#pragma unroll
    for (int i = 0; i < AI; ++i) {
      const int it = threadIdx.x + 256 * i, row = it / 16;
      *reinterpret_cast<bf16x8 *>(sa[buf] + (row >> 5) * G::ROW_ELEMS + G::row_off(row & 31, it % 16)) =
          r.missing >> i & 1u ? zero8() : r.v[i];
    }
    __syncthreads();  // (the other buffer was last read before this barrier)
    o = o1;
    o1 = next(o1);
    if (AHEAD)
#pragma unroll
      for (int ks = 0; ks < C / 32; ++ks) fetch_weights(min(o, 26), ks, nxt);
    fetch_rows(AHEAD ? o1 : o, r);
#pragma unroll
    for (int ks = 0; ks < C / 32; ++ks) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const bf16x8 av = lds_row_operand<C>(sa[buf] + (mt >> 1) * G::ROW_ELEMS, mt & 1, ks);
        acc[mt][0] = mfma16(av, cur.v[0][ks], acc[mt][0]);
        acc[mt][1] = mfma16(av, cur.v[1][ks], acc[mt][1]);
      }
      if (!AHEAD) fetch_weights(min(o, 26), ks, nxt);
    }
  };
  if (o < 27) {
    fetch_rows(o, ra);
    if (AHEAD) fetch_rows(o1, rb);
#pragma unroll
    for (int ks = 0; ks < C / 32; ++ks) fetch_weights(o, ks, wa);
    Weights &w1 = AHEAD ? wb : wa;
    Rows &r1 = AHEAD ? rb : ra;
    while (true) {
      step(0, wa, w1, ra);
      if (o >= 27) break;
      step(1, w1, wa, r1);
      if (o >= 27) break;
    }
  }
  float *out = cs.out + blockIdx.y * part_stride;
  // lane: column n of half a -> channel 32*wid + 8*(n >> 2) + 4*a + (n & 3); rows 4*quad + i of tile mt -> token
  // pos0 + 32*(mt >> 1) + 8*quad + 4*(mt & 1) + i
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int ch = wrow + 4 * a;
    const float bs = cs.bias && blockIdx.y == 0 ? bf16_to_f32(cs.bias[ch]) : 0.f;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = pos0 + 32 * (mt >> 1) + 8 * quad + 4 * (mt & 1) + i;
        if (t < N) out[(size_t)t * C + ch] = acc[mt][a][i] + bs;
      }
  }
}

// Mean over the tokens of each compression block (contiguous in sorted order); one workgroup per block.
// A token's row is the sum of P rows part_stride apart, in order.
template <int P>
__global__ void c_pool(Pair<const float *> Ys, size_t part_stride, const int32_t *__restrict__ cmp_start, int C, Pair<bf16_t *> xcs) {
  const float *__restrict__ Y = Ys.v[blockIdx.z];
  const int c = blockIdx.x, b = cmp_start[c], e = cmp_start[c + 1];
  const float inv = 1.0f / (float)(e - b);  // same arithmetic as the plain mean pool of the attention path
  for (int f = threadIdx.x; f < C; f += blockDim.x) {
    float s = 0.f;
    for (int pos = b; pos < e; pos += 8) {  // eight tokens in flight, those past the end again the last; the order of the additions stays
      float v[P][8];
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int u = 0; u < 8; ++u) v[p][u] = Y[p * part_stride + (size_t)min(pos + u, e - 1) * C + f];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        float x = v[0][u];
#pragma unroll
        for (int p = 1; p < P; ++p) x += v[p][u];
        if (pos + u < e) s += x;
      }
    }
    xcs.v[blockIdx.z][(size_t)c * C + f] = f32_to_bf16(s * inv);
  }
}

// dY[pos] = dXc[block(pos)] / count(block)   (bf16, sorted order): gradient of the mean pool.  The workgroups behind those:
// dbias[f] = sum over blocks of dXc[c][f]  (the pool's 1/count and the block's count cancel): partial sums over
// DBIAS_PARTS row ranges, added in order by c_sum_last.
constexpr int DBIAS_PARTS = 32;
__global__ __launch_bounds__(256) void c_expand(Pair<const float *> dxcs, const int32_t *__restrict__ tok_cmp, const int32_t *__restrict__ cmp_start,
                                                int N, int Nc, int C, Pair<bf16_t *> dYs, Pair<float *> parts) {
  const float *__restrict__ dxc = dxcs.v[blockIdx.z];
  const unsigned expand_wgs = gridDim.x - DBIAS_PARTS;
  if (blockIdx.x >= expand_wgs) {
    const int part = (int)(blockIdx.x - expand_wgs), per = (Nc + DBIAS_PARTS - 1) / DBIAS_PARTS;
    const int b = min(Nc, part * per), e = min(Nc, b + per), f = threadIdx.x;
    if (f >= C) return;  // C <= 256
    float s = 0.f;
#pragma unroll 8
    for (int c = b; c < e; ++c) s += dxc[(size_t)c * C + f];
    parts.v[blockIdx.z][(size_t)part * C + f] = s;
    return;
  }
  bf16_t *__restrict__ dY = dYs.v[blockIdx.z];
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  const int per = C / 8;
  if (i >= (size_t)N * per) return;
  const int pos = (int)(i / per), c0 = (int)(i % per) * 8;
  const int c = tok_cmp[pos];
  const float inv = 1.0f / (float)(cmp_start[c + 1] - cmp_start[c]);
  bf16x8 r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r[j] = (__bf16)(dxc[(size_t)c * C + c0 + j] * inv);
  *reinterpret_cast<bf16x8 *>(dY + (size_t)pos * C + c0) = r;
}

// dx[perm[pos]] += dU[pos]   (caller order, parameter dtype)
__global__ void c_dx_accum(Pair<float *> dUs, int parts, size_t part_stride, const int32_t *__restrict__ perm, int N, int C, Pair<bf16_t *> dxs) {
  float *__restrict__ dU = dUs.v[blockIdx.z];
  bf16_t *dx = dxs.v[blockIdx.z];
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int per = C / 8;
  if (i >= (size_t)N * per) return;
  const int pos = (int)(i / per), c0 = (int)(i % per) * 8;
  bf16_t *d = dx + (size_t)perm[pos] * C + c0;
  const bf16x8 cur = ld8(d);
  float *row = dU + (size_t)pos * C + c0, v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = row[j];
  if (parts > 1) {  // the rows of the parts, in order, and their sum for what reads it next
    for (int p = 1; p < parts; ++p)
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] += row[p * part_stride + j];
#pragma unroll
    for (int j = 0; j < 8; ++j) row[j] = v[j];
  }
  bf16x8 r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r[j] = (__bf16)((float)cur[j] + v[j]);
  *reinterpret_cast<bf16x8 *>(d) = r;
}

// dPE, first stage: the tokens of chunk blockIdx.x are visited in order, thread f owns channel f of every table row
// (LDS [m^3][C] fp32), so no two threads ever add to the same cell.
__global__ void c_dpe_partial(Pair<const float *> dUs, const uint64_t *__restrict__ keys, int N, int C, int bits, int m,
                              int chunk, Pair<float *> parts) {
  extern __shared__ __align__(16) float tbl[];
  const float *__restrict__ dU = dUs.v[blockIdx.z];
  float *__restrict__ part = parts.v[blockIdx.z];
  const int rows = m * m * m;
  for (int i = threadIdx.x; i < rows * C / 4; i += blockDim.x) reinterpret_cast<float4 *>(tbl)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  __syncthreads();
  const int b = blockIdx.x * chunk, e = min(N, b + chunk);
  for (int p0 = b; p0 < e; p0 += 16) {  // sixteen tokens' rows in flight, added in token order
    int row[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const Site s = decode(keys[min(p0 + u, e - 1)], bits);
      row[u] = (((s.x & (m - 1)) * m + (s.y & (m - 1))) * m + (s.z & (m - 1))) * C;
    }
    for (int f = threadIdx.x; f < C; f += blockDim.x) {
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = dU[(size_t)min(p0 + u, e - 1) * C + f];
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (p0 + u < e) tbl[row[u] + f] += v[u];
    }
  }
  __syncthreads();
  float4 *to = reinterpret_cast<float4 *>(part + (size_t)blockIdx.x * rows * C);
  for (int i = threadIdx.x; i < rows * C / 4; i += blockDim.x) to[i] = reinterpret_cast<const float4 *>(tbl)[i];
}

// Ordered sums of partial results.  c_sum_parts: out[g][i] = sum of part[g*group + j][i], j = 0 .. group-1 (parts past n_parts are
// skipped), which keeps the work parallel where there are many.  c_sum_last: the totals of the three parameter gradients in one
// launch, workgroups one after the other.  The order of the additions is fixed either way.
__device__ inline float sum_in_order(const float *part, size_t len, int b, int e) {
  float s = 0.f;
#pragma unroll 8
  for (int k = b; k < e; ++k) s += part[(size_t)k * len];
  return s;
}
__global__ void c_sum_parts(Pair<const float *> parts, int n_parts, int n_groups, size_t len, Pair<float *> outs) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= len) return;
  const int group = (n_parts + n_groups - 1) / n_groups;
  const int g = blockIdx.y, b = g * group;
  outs.v[blockIdx.z][(size_t)g * len + i] = sum_in_order(parts.v[blockIdx.z] + i, len, b, min(n_parts, b + group));
}
struct SumJob {
  Pair<const float *> parts;
  Pair<float *> outs;
  int n_parts;
  unsigned len;
  __host__ __device__ unsigned wgs() const { return (len + 255) / 256; }
};
struct SumJobs { SumJob j[3]; };
__global__ __launch_bounds__(256) void c_sum_last(SumJobs jobs) {
  unsigned wg = blockIdx.x;
  int d = 0;
  while (d < 2 && wg >= jobs.j[d].wgs()) wg -= jobs.j[d].wgs(), ++d;
  const SumJob &j = jobs.j[d];
  const unsigned i = wg * 256 + threadIdx.x;
  if (i < j.len) j.outs.v[blockIdx.z][i] = sum_in_order(j.parts.v[blockIdx.z] + i, j.len, 0, j.n_parts);
}

// Weight gradient: dW[o][ci][co] = sum_pos U[nbr[pos][o]][ci] * dY[pos][co], a contraction over tokens.  A workgroup
// takes one offset, one chunk of tokens and one CT x CT tile of the C x C matrix.  The tokens of a segment that have a
// neighbour at the offset are listed first (in order, by ballots): on a surface that is about half of them, and the others
// add nothing.  32-row tiles of the listed U and dY rows go through LDS row-major (two buffers, one barrier per tile, the
// next tile's rows in flight), both MFMA operands are transposing LDS reads of them.  Wave w owns the 16-row blocks w, w+4,
// .. of the tile.
// Bound: latency of the gathers, so 1024 tokens per workgroup where that fills the chip (see mod_plan).  Keys and values of
// 10.7 k tokens: 180 us (every token multiplied, loads not ahead of the products) -> 38 us; the whole module forward,
// twice forward and once backward in a layer's training step: 2430 -> 1903 us of the step.
constexpr int DW_SEG = 1024;  // tokens listed at a time
template <int CT>
__global__ __launch_bounds__(256) void c_dw(Pair<const bf16_t *> Us, Pair<const bf16_t *> dYs,
                                            const int32_t *__restrict__ nbr, int N, int C, int chunk, Pair<float *> parts) {
  using G = TileGeom<CT>;
  __shared__ __align__(16) bf16_t su[2][G::ROW_ELEMS], sy[2][G::ROW_ELEMS];
  __shared__ int2 list[DW_SEG];           // (neighbour, token)
  __shared__ int count[DW_SEG / 256][4];  // listed tokens per round and wavefront
  const int tiles = C / CT, zt = (int)blockIdx.z % (tiles * tiles), src = (int)blockIdx.z / (tiles * tiles);
  const bf16_t *__restrict__ U = Us.v[src], *__restrict__ dY = dYs.v[src];
  const int o = blockIdx.x, s = blockIdx.y;
  const int ci0 = (zt / tiles) * CT, co0 = (zt % tiles) * CT;
  const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, quad = lane >> 4;
  constexpr int MB = CT / 16 / 4 > 0 ? CT / 16 / 4 : 1;  // 16-row blocks per wave
  constexpr int NBK = CT / 16;
  constexpr int NI = G::ROW_ITEMS > 256 ? G::ROW_ITEMS / 256 : 1, SEGS = CT / 8;  // 16-byte items per thread and tile
  const bool wave_on = wid < CT / 16, stages = (int)threadIdx.x < G::ROW_ITEMS;
  f32x4 acc[MB][NBK];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int nb = 0; nb < NBK; ++nb) acc[a][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int b = s * chunk, e = min(N, b + chunk);
  int buf = 0;
  for (int s0 = b; s0 < e; s0 += DW_SEG) {
    int nb_of[DW_SEG / 256];
    uint64_t has[DW_SEG / 256];
#pragma unroll
    for (int r = 0; r < DW_SEG / 256; ++r) {
      const int pos = s0 + 256 * r + (int)threadIdx.x;
      nb_of[r] = pos < e ? nbr[(size_t)pos * 27 + o] : -1;
    }
#pragma unroll
    for (int r = 0; r < DW_SEG / 256; ++r) {
      has[r] = __ballot(nb_of[r] >= 0);
      if (lane == 0) count[r][wid] = __popcll(has[r]);
    }
    __syncthreads();  // (the list of the segment before was last read before its last barrier)
    int total = 0;
#pragma unroll
    for (int r = 0; r < DW_SEG / 256; ++r)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if (w == wid && nb_of[r] >= 0)
          list[total + __popcll(has[r] & ((1ull << lane) - 1ull))] = make_int2(nb_of[r], s0 + 256 * r + (int)threadIdx.x);
        total += count[r][w];
      }
    __syncthreads();
    bf16x8 xu[NI], xy[NI];
    auto fetch = [&](int t0) {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int it = threadIdx.x + 256 * i, row = t0 + it / SEGS, seg = it % SEGS;
        xu[i] = xy[i] = zero8();
        if (stages && row < total) {
          const int2 l = list[row];
          xu[i] = ld8(U + (size_t)l.x * C + ci0 + 8 * seg);
          xy[i] = ld8(dY + (size_t)l.y * C + co0 + 8 * seg);
        }
      }
    };
    fetch(0);
    for (int t0 = 0; t0 < total; t0 += 32, buf ^= 1) {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int it = threadIdx.x + 256 * i;
        if (stages) {
          *reinterpret_cast<bf16x8 *>(su[buf] + G::row_off(it / SEGS, it % SEGS)) = xu[i];
          *reinterpret_cast<bf16x8 *>(sy[buf] + G::row_off(it / SEGS, it % SEGS)) = xy[i];
        }
      }
      __syncthreads();  // (the other buffer was last read before this barrier)
      if (t0 + 32 < total) fetch(t0 + 32);
      if (wave_on) {
        bf16x8 av[MB];
#pragma unroll
        for (int a = 0; a < MB; ++a) av[a] = lds_tr_operand<CT>(su[buf], wid + 4 * a);
#pragma unroll
        for (int nb = 0; nb < NBK; ++nb) {
          const bf16x8 bv = lds_tr_operand<CT>(sy[buf], nb);
#pragma unroll
          for (int a = 0; a < MB; ++a) acc[a][nb] = mfma16(av[a], bv, acc[a][nb]);
        }
      }
    }
  }
  if (!wave_on) return;
  // C layout: lane holds column co = 16*nb + n, rows ci = 16*(wid + 4a) + 4*quad + i
  float *dst = parts.v[src] + ((size_t)s * 27 + o) * C * C;
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int nb = 0; nb < NBK; ++nb)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        dst[(size_t)(ci0 + 16 * (wid + 4 * a) + 4 * quad + i) * C + co0 + 16 * nb + n] = acc[a][nb][i];
}

constexpr int PE_GROUPS = 32;  // first-level groups of the ordered dPE sum

// The convolution of n tensors of 128 channels: tokens per workgroup, and parts that a tile's offsets are dealt out to, a workgroup
// each; the kernel that reads the result adds them.  128 tokens per workgroup read the weights half as often, 64 fill the chip
// while 256 workgroups of 64 do not (keys and values, 64 against 128 tokens: 123 and 123 us at 10.7 k, 162 and 136 at 17 k).  A
// tile's offsets are a serial chain and a compute unit holds two workgroups, so parts are taken while all of them run at once:
// the module of keys and values, one -> three parts, forward and backward: 1 k tokens 110 and 106 -> 79 and 92 us, 3 k 112 and 111 ->
// 102 and 106, 10.7 k (tiles of 128) 180 and 163 -> 143 and 149; two parts at 14 k 187 and 172 -> 156 and 163.  Two parts of 64
// tokens save less of the short chain than the second set of rows costs: 5.5 k 121 and 119 -> 126 and 124, 8 k 127 and 126 -> 133 and 133.
// The parts are 32-bit rows added in order, another order of the same sum than one chain over the offsets: at 8 sizes of 0.7 to 30 k tokens the
// 2-norm error of pooled rows and dx (bf16) against 64 bits is the same to 8 digits, that of the PE gradient, a 32-bit sum of dU, 21 to 39 % smaller.
struct ConvShape { int tok, parts; };
ConvShape conv_shape(int N, int C, int n) {
  if (C != 128) return {0, 1};
  const int tok = (long long)N * n > 16384 ? 128 : 64;
  const long long wgs = (long long)((N + tok - 1) / tok) * n;
  const int parts = 3 * wgs <= 512 ? 3 : 2 * wgs <= 512 && tok == 128 ? 2 : 1;
  return {tok, parts};
}

// Workspace of a pass over n tensors; per-tensor arrays lie one after the other.  The inputs (neighbour table and U) have a
// region of their own: a backward pass that follows a recomputed forward pass finds them there.
struct ModPlan {
  size_t nbr, u, inputs_total;
  size_t wt, y, dy, du, pw, ppe, ppe2, pb, total;
  size_t rows16, rows32, wlen, plen;  // bytes per tensor of [N][C] bf16 / fp32; elements of the weights and of the PE table
  int dw_chunks, dw_chunk, pe_chunks, pe_chunk;
};

ModPlan mod_plan(int N, int C, int m, int n, bool backward) {
  ModPlan p{};
  size_t off = 0;
  auto take = [&](size_t b) { size_t r = off; off += align_up(b, 256); return r; };
  p.rows16 = align_up((size_t)N * C * 2, 256);
  p.rows32 = align_up((size_t)N * C * 4, 256);
  p.wlen = (size_t)27 * C * C;
  p.plen = (size_t)m * m * m * C;
  p.nbr = take((size_t)N * 27 * 4);
  p.u = take(n * p.rows16);
  p.inputs_total = off;
  off = 0;
  if (!backward) {
    p.wt = take(n * p.wlen * 2);
    p.y = take(n * p.rows32 * conv_shape(N, C, n).parts);
  } else {
    p.dy = take(n * p.rows16);
    p.du = take(n * p.rows32 * conv_shape(N, C, n).parts);
    // a chunk is a workgroup per offset: 1024 tokens of a small problem fill the chip, 32 chunks bound the partial sums
    p.dw_chunks = N > 0 ? (N + 1023) / 1024 : 1;
    if (p.dw_chunks > 32) p.dw_chunks = 32;
    p.dw_chunk = ((N + p.dw_chunks - 1) / p.dw_chunks + 31) / 32 * 32;
    if (p.dw_chunk < 32) p.dw_chunk = 32;
    p.pw = take(n * p.dw_chunks * p.wlen * 4);
    p.pe_chunks = N > 0 ? (N + 63) / 64 : 1;
    if (p.pe_chunks > 1024) p.pe_chunks = 1024;
    p.pe_chunk = (N + p.pe_chunks - 1) / p.pe_chunks;
    if (p.pe_chunk < 1) p.pe_chunk = 1;
    p.ppe = take(n * p.pe_chunks * p.plen * 4);
    p.ppe2 = take(n * PE_GROUPS * p.plen * 4);
    p.pb = take((size_t)n * DBIAS_PARTS * C * 4);
  }
  p.total = off;
  return p;
}

int check(const ssa_params_t *p, const ssa_blocks_t *b, int *C) {
  if (!p || !b) return SSA_ERR_NULL;
  if (p->n_tokens != b->N || p->n_batch != b->B || p->grid != b->G || p->m_cmp != b->m_cmp) return SSA_ERR_MISMATCH;
  if (p->n_heads_kv < 1 || p->head_dim < 1) return SSA_ERR_BAD_HEADS;
  if (p->dtype != SSA_BF16 || b->dims != 3) return SSA_ERR_UNSUPPORTED;  // the convolution is defined on the voxel grid
  const long long c = (long long)p->n_heads_kv * p->head_dim;
  if (c != 32 && c != 64 && c != 128 && c != 256) return SSA_ERR_UNSUPPORTED;
  if ((size_t)p->m_cmp * p->m_cmp * p->m_cmp * (size_t)c * 4 > 64 * 1024) return SSA_ERR_UNSUPPORTED;
  if ((long long)p->n_tokens * c >= (1ll << 31)) return SSA_ERR_BAD_SHAPE;
  *C = (int)c;
  return SSA_OK;
}

template <bool MIRROR>
void launch_conv(int C, const Pair<ConvSrc> &src, int n, const int32_t *nbr, int N, ConvShape shape, size_t part_stride, hipStream_t s) {
  // 64 tokens per wavefront and up to 128 output channels per workgroup row (blockIdx.y picks the channel range)
  const dim3 grid((unsigned)((N + 255) / 256), (unsigned)(C > 128 ? C / 128 : 1), n);
  switch (C) {
    case 32: c_conv<32, MIRROR, 4, 2><<<grid, 256, 0, s>>>(src, nbr, N); break;
    case 64: c_conv<64, MIRROR, 4, 4><<<grid, 256, 0, s>>>(src, nbr, N); break;
    case 128:
      if (shape.tok == 128) c_conv128<MIRROR, 128><<<dim3((unsigned)((N + 127) / 128), shape.parts, n), 256, 0, s>>>(src, nbr, N, part_stride);
      else c_conv128<MIRROR, 64><<<dim3((unsigned)((N + 63) / 64), shape.parts, n), 256, 0, s>>>(src, nbr, N, part_stride);
      break;
    default: c_conv<256, MIRROR, 4, 8><<<grid, 256, 0, s>>>(src, nbr, N); break;
  }
}

// A Pair of pointers, `stride` bytes apart, into a workspace.
template <class T>
Pair<T *> carve(char *ws, size_t off, size_t stride) {
  return Pair<T *>{{(T *)(ws + off), (T *)(ws + off + stride)}};
}
template <class T>
Pair<const T *> as_const(const Pair<T *> &p) { return Pair<const T *>{{p.v[0], p.v[1]}}; }

// Neighbour table and U of the n tensors; wt: their transposed weights go there, or {null, null}.
void prepare_inputs(const ssa_blocks_t *b, int C, int n, const CmpTensor *t, const ModPlan &pl, char *in, Pair<bf16_t *> wt, hipStream_t s) {
  PrepareArgs a{b->sorted_keys, b->item_start, b->perm, b->N, b->G, b->bits, C, b->m_cmp, (int32_t *)(in + pl.nbr)};
  a.U = carve<bf16_t>(in, pl.u, pl.rows16);
  a.wt = wt;
  for (int i = 0; i < 2; ++i) {
    const CmpTensor &x = t[i < n ? i : n - 1];
    a.x.v[i] = (const bf16_t *)x.x;
    a.pe.v[i] = (const bf16_t *)x.w->pe;
    a.w.v[i] = (const bf16_t *)x.w->w;
  }
  a.nbr_wgs = (unsigned)(((size_t)b->N * 27 + 255) / 256);
  a.pe_wgs = (unsigned)(((size_t)b->N * (C / 8) + 255) / 256);
  a.wt_wgs = wt.v[0] ? (unsigned)((pl.wlen + 255) / 256) : 0u;
  c_prepare<<<a.nbr_wgs + n * (a.pe_wgs + a.wt_wgs), 256, 0, s>>>(a);
}

}  // namespace

size_t cmp_module_workspace(const ssa_params_t *p, const ssa_blocks_t *b, int n, bool backward) {
  int C;
  if (check(p, b, &C) != SSA_OK) return 0;
  return mod_plan(b->N, C, b->m_cmp, n, backward).total + 256;
}
size_t cmp_module_input_bytes(const ssa_params_t *p, const ssa_blocks_t *b, int n) {
  int C;
  if (check(p, b, &C) != SSA_OK) return 0;
  return mod_plan(b->N, C, b->m_cmp, n, false).inputs_total + 256;
}

// n = 1 or 2 tensors; the arguments are checked and N > 0.
int cmp_module_forward(const ssa_params_t *p, const ssa_blocks_t *b, int n, const CmpTensor *t, void *in_, void *ws_, hipStream_t s) {
  const int N = b->N, C = p->n_heads_kv * p->head_dim;
  const ModPlan pl = mod_plan(N, C, b->m_cmp, n, false);
  char *in = (char *)align_up((size_t)in_, 256), *ws = (char *)align_up((size_t)ws_, 256);
  const Pair<bf16_t *> U = carve<bf16_t>(in, pl.u, pl.rows16), Wt = carve<bf16_t>(ws, pl.wt, pl.wlen * 2);
  const Pair<float *> Y = carve<float>(ws, pl.y, pl.rows32);
  ProfScope ps(PROF_CMP_MODULE, s);
  prepare_inputs(b, C, n, t, pl, in, Wt, s);
  Pair<ConvSrc> src{};
  for (int i = 0; i < n; ++i) src.v[i] = ConvSrc{U.v[i], Wt.v[i], (const bf16_t *)t[i].w->bias, Y.v[i]};
  const ConvShape shape = conv_shape(N, C, n);
  const size_t part_stride = n * pl.rows32 / 4;
  launch_conv<false>(C, src, n, (const int32_t *)(in + pl.nbr), N, shape, part_stride, s);
  auto pool = [&](auto kernel) {
    kernel<<<dim3(b->Nc, 1, n), 128, 0, s>>>(as_const(Y), part_stride, b->cmp_start, C, Pair<bf16_t *>{{(bf16_t *)t[0].xc, (bf16_t *)t[n - 1].xc}});
  };
  shape.parts == 1 ? pool(c_pool<1>) : shape.parts == 2 ? pool(c_pool<2>) : pool(c_pool<3>);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}

// prepared: the input region holds the neighbour table and U of these tensors from cmp_module_forward on the same n.
int cmp_module_backward(const ssa_params_t *p, const ssa_blocks_t *b, int n, const CmpTensor *t, bool prepared, void *in_, void *ws_,
                        hipStream_t s) {
  const int N = b->N, m = b->m_cmp, C = p->n_heads_kv * p->head_dim;
  const ModPlan pl = mod_plan(N, C, m, n, true);
  char *in = (char *)align_up((size_t)in_, 256), *ws = (char *)align_up((size_t)ws_, 256);
  const int32_t *nbr = (const int32_t *)(in + pl.nbr);
  const Pair<bf16_t *> U = carve<bf16_t>(in, pl.u, pl.rows16), dY = carve<bf16_t>(ws, pl.dy, pl.rows16);
  const Pair<float *> dU = carve<float>(ws, pl.du, pl.rows32), pw = carve<float>(ws, pl.pw, pl.dw_chunks * pl.wlen * 4);
  const Pair<float *> ppe = carve<float>(ws, pl.ppe, pl.pe_chunks * pl.plen * 4), ppe2 = carve<float>(ws, pl.ppe2, PE_GROUPS * pl.plen * 4);
  const Pair<float *> pb = carve<float>(ws, pl.pb, (size_t)DBIAS_PARTS * C * 4);
  const Pair<const float *> dxc{{t[0].dxc, t[n - 1].dxc}};
  ProfScope ps(PROF_CMP_MODULE_BWD, s);
  if (!prepared) prepare_inputs(b, C, n, t, pl, in, Pair<bf16_t *>{}, s);
  const size_t items = (size_t)N * (C / 8);
  const dim3 igrid((unsigned)((items + 255) / 256), 1, n);
  c_expand<<<dim3(igrid.x + DBIAS_PARTS, 1, n), 256, 0, s>>>(dxc, b->tok_cmp, b->cmp_start, N, b->Nc, C, dY, pb);
  // data gradient: dU[pos] = sum_o dY[token that took pos as neighbour o] * w[o]^T; w as given has c_out contiguous
  Pair<ConvSrc> src{};
  for (int i = 0; i < n; ++i) src.v[i] = ConvSrc{dY.v[i], (const bf16_t *)t[i].w->w, nullptr, dU.v[i]};
  const ConvShape shape = conv_shape(N, C, n);
  const size_t part_stride = n * pl.rows32 / 4;
  launch_conv<true>(C, src, n, nbr, N, shape, part_stride, s);
  c_dx_accum<<<igrid, 256, 0, s>>>(dU, shape.parts, part_stride, b->perm, N, C, Pair<bf16_t *>{{(bf16_t *)t[0].dx, (bf16_t *)t[n - 1].dx}});
  const unsigned pgrid = (unsigned)((pl.plen + 255) / 256);
  c_dpe_partial<<<dim3(pl.pe_chunks, 1, n), 128, pl.plen * 4, s>>>(as_const(dU), b->sorted_keys, N, C, b->bits, m, pl.pe_chunk, ppe);
  c_sum_parts<<<dim3(pgrid, PE_GROUPS, n), 256, 0, s>>>(as_const(ppe), pl.pe_chunks, PE_GROUPS, pl.plen, ppe2);
  const int CT = C < 128 ? C : 128;
  const dim3 g(27, pl.dw_chunks, (C / CT) * (C / CT) * n);
  switch (CT) {
    case 32: c_dw<32><<<g, 256, 0, s>>>(as_const(U), as_const(dY), nbr, N, C, pl.dw_chunk, pw); break;
    case 64: c_dw<64><<<g, 256, 0, s>>>(as_const(U), as_const(dY), nbr, N, C, pl.dw_chunk, pw); break;
    default: c_dw<128><<<g, 256, 0, s>>>(as_const(U), as_const(dY), nbr, N, C, pl.dw_chunk, pw); break;
  }
  const SumJobs last{{{as_const(pw), Pair<float *>{{t[0].dw, t[n - 1].dw}}, pl.dw_chunks, (unsigned)pl.wlen},
                      {as_const(ppe2), Pair<float *>{{t[0].dpe, t[n - 1].dpe}}, PE_GROUPS, (unsigned)pl.plen},
                      {as_const(pb), Pair<float *>{{t[0].dbias, t[n - 1].dbias}}, DBIAS_PARTS, (unsigned)C}}};
  c_sum_last<<<dim3(last.j[0].wgs() + last.j[1].wgs() + last.j[2].wgs(), 1, n), 256, 0, s>>>(last);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}

// Argument checks of the public calls on one tensor (backward: the gradients too).
int cmp_module_check(const CmpTensor &t, bool backward) {
  if (!t.x || !t.w || !t.w->pe || !t.w->w || !t.w->bias) return SSA_ERR_NULL;
  if (!backward) {
    if (!t.xc) return SSA_ERR_NULL;
    return aligned16(t.x, t.w->pe, t.w->w, t.w->bias, t.xc) ? SSA_OK : SSA_ERR_ALIGNMENT;
  }
  if (!t.dxc || !t.dx || !t.dpe || !t.dw || !t.dbias) return SSA_ERR_NULL;
  return aligned16(t.x, t.w->pe, t.w->w, t.w->bias, t.dxc, t.dx, t.dpe, t.dw, t.dbias) ? SSA_OK : SSA_ERR_ALIGNMENT;
}

extern "C" size_t ssa_compress_workspace_bytes(const ssa_params_t *p, const ssa_blocks_t *b, int for_backward) {
  const size_t n = cmp_module_workspace(p, b, 1, for_backward != 0);
  return n == 0 ? 0 : n + cmp_module_input_bytes(p, b, 1);
}

extern "C" int ssa_compress_forward(const ssa_params_t *p, const ssa_blocks_t *b, const void *x,
                                    const ssa_cmp_weights_t *wts, void *x_cmp, void *ws, size_t ws_bytes, void *stream) {
  int C;
  int rc = check(p, b, &C);
  if (rc != SSA_OK) return rc;
  if (b->N == 0) return SSA_OK;
  CmpTensor t{};
  t.x = x; t.w = wts; t.xc = x_cmp;
  rc = cmp_module_check(t, false);
  if (rc != SSA_OK) return rc;
  if (!ws || ws_bytes < ssa_compress_workspace_bytes(p, b, 0)) return SSA_ERR_WORKSPACE;
  return cmp_module_forward(p, b, 1, &t, ws, (char *)ws + cmp_module_input_bytes(p, b, 1), (hipStream_t)stream);
}

extern "C" int ssa_compress_backward(const ssa_params_t *p, const ssa_blocks_t *b, const void *x,
                                     const ssa_cmp_weights_t *wts, const float *dx_cmp, void *dx_accum, float *dpe,
                                     float *dw, float *dbias, void *ws, size_t ws_bytes, void *stream) {
  int C;
  int rc = check(p, b, &C);
  if (rc != SSA_OK) return rc;
  hipStream_t s = (hipStream_t)stream;
  if (b->N == 0) {  // no tokens: the parameter gradients are zero
    if (!dpe || !dw || !dbias) return SSA_ERR_NULL;
    const size_t plen0 = (size_t)b->m_cmp * b->m_cmp * b->m_cmp * C, wlen0 = (size_t)27 * C * C;
    const Pair<const float *> none{};
    c_sum_parts<<<(unsigned)((plen0 + 255) / 256), 256, 0, s>>>(none, 0, 1, plen0, Pair<float *>{{dpe, dpe}});
    c_sum_parts<<<(unsigned)((wlen0 + 255) / 256), 256, 0, s>>>(none, 0, 1, wlen0, Pair<float *>{{dw, dw}});
    c_sum_parts<<<(C + 255) / 256, 256, 0, s>>>(none, 0, 1, (size_t)C, Pair<float *>{{dbias, dbias}});
    return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
  }
  CmpTensor t{};
  t.x = x; t.w = wts; t.dxc = dx_cmp; t.dx = dx_accum; t.dpe = dpe; t.dw = dw; t.dbias = dbias;
  rc = cmp_module_check(t, true);
  if (rc != SSA_OK) return rc;
  if (!ws || ws_bytes < ssa_compress_workspace_bytes(p, b, 1)) return SSA_ERR_WORKSPACE;
  return cmp_module_backward(p, b, 1, &t, false, ws, (char *)ws + cmp_module_input_bytes(p, b, 1), s);
}
