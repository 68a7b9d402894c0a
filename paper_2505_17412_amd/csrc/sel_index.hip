// Inverse of the selection (gfx950): for every (KV head, selection block) the ascending list of sorted positions of the
// query tokens whose row of the index tensor I (Algorithm 1) holds the block, each with its rank in that row, and the cuts
// of every list into work chunks.  The block-centric selection kernels (forward and dQ) and the key-centric dK/dV kernel
// walk these lists.  A counting sort over tiles of POS_TILE sorted positions: a tile's selections are marked in a bit
// matrix in LDS (integer OR: order independent), so that the population count below a bit is the entry's rank inside its
// tile; per-tile counts are turned into offsets, and every entry then writes itself to its final place.  Integer work
// only, and the lists do not depend on scheduling.
// Bound: latency of five small dependent launches (every pass reads or writes a few MB), so a tile is small enough that all
// its loads are in flight at once.  62k tokens, top-16, 2 KV heads: 59 us (146 us with a bit matrix in memory, whose
// passes had one workgroup per 1024 positions); 2k tokens, top-8: 24 us (45 us).
#include "mfma_launch.h"

namespace {

constexpr int POS_TILE = 256;              // sorted positions per tile (8 words of 32 bits per key)
constexpr int TILE_WORDS = POS_TILE / 32;
constexpr int KEY_TILE = 2048;             // selection blocks of one KV head a workgroup covers: 64 KB of bits
constexpr int SEL_THREADS = 512;

struct SelArgs {
  const int32_t *idx, *perm;
  int N, Hkv, T, Ns;
};

__device__ inline int sel_block(const SelArgs &a, int p0, int npos, int g, int e) {  // block of entry e of the tile, or -1
  const int pl = e / a.T, j = e - pl * a.T;
  return pl < npos ? a.idx[((size_t)a.perm[p0 + pl] * a.Hkv + g) * a.T + j] : -1;
}

// Pass 1: entries per (key, tile).  cnt[key][n_tiles].  Workgroup (0,0,0) also clears the chunk-order counters.
__global__ __launch_bounds__(SEL_THREADS) void m_sel_count(SelArgs a, int n_tiles, uint32_t *__restrict__ cnt,
                                                           uint32_t *__restrict__ bins, int bins_stride, int n_bins) {
  extern __shared__ __align__(16) uint32_t sel_bits[];  // [nb][TILE_WORDS]
  const int tile = blockIdx.x, g = blockIdx.y, b0 = blockIdx.z * KEY_TILE, nb = min(KEY_TILE, a.Ns - b0);
  if (g == 0 && blockIdx.z == 0)
    for (int i = tile * SEL_THREADS + threadIdx.x; i < n_bins; i += n_tiles * SEL_THREADS) bins[i] = bins[bins_stride + i] = 0u;
  for (int i = threadIdx.x; i < nb * TILE_WORDS; i += SEL_THREADS) sel_bits[i] = 0u;
  __syncthreads();
  const int p0 = tile * POS_TILE, npos = min(POS_TILE, a.N - p0), ne = npos * a.T;
  for (int e0 = 0; e0 < ne; e0 += 8 * SEL_THREADS) {
    int b[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) b[u] = sel_block(a, p0, npos, g, e0 + u * SEL_THREADS + threadIdx.x);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int pl = (e0 + u * SEL_THREADS + (int)threadIdx.x) / a.T;
      if ((unsigned)(b[u] - b0) < (unsigned)nb) atomicOr(&sel_bits[(b[u] - b0) * TILE_WORDS + (pl >> 5)], 1u << (pl & 31));
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nb; i += SEL_THREADS) {
    const uint4 x = *reinterpret_cast<const uint4 *>(sel_bits + i * TILE_WORDS), y = *reinterpret_cast<const uint4 *>(sel_bits + i * TILE_WORDS + 4);
    cnt[((size_t)g * a.Ns + b0 + i) * n_tiles + tile] = __popc(x.x) + __popc(x.y) + __popc(x.z) + __popc(x.w) + __popc(y.x) + __popc(y.y) + __popc(y.z) + __popc(y.w);
  }
}

// Pass 2: per key (one wavefront each) the exclusive prefix of its counts over the tiles, in place, and their sum.
__global__ __launch_bounds__(256) void m_sel_scan_tiles(uint32_t *__restrict__ cnt, int n_keys, int n_tiles, uint32_t *__restrict__ counts) {
  const int key = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (key >= n_keys) return;
  uint32_t *row = cnt + (size_t)key * n_tiles;
  uint32_t carry = 0;
  for (int t0 = 0; t0 < n_tiles; t0 += 256) {  // four tiles per lane and round
    uint32_t v[4], own = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = t0 + lane * 4 + u;
      v[u] = t < n_tiles ? row[t] : 0u;
      own += v[u];
    }
    uint32_t incl = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t o = __shfl_up(incl, off);
      if (lane >= off) incl += o;
    }
    uint32_t run = carry + incl - own;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = t0 + lane * 4 + u;
      if (t < n_tiles) row[t] = run;
      run += v[u];
    }
    carry += __shfl(incl, 63);
  }
  if (lane == 0) counts[key] = carry;
}

// Pass 3, single workgroup: from the per-(g, block) selector counts, four exclusive prefix sums over the n keys:
// start (list offsets), chunk_start (work chunks of chunk_len query tokens), part_row_start (rows of partial sums:
// chunks x keys of the block), bc_chunk_start (work chunks of bc_chunk_len query tokens).
__global__ __launch_bounds__(1024) void m_scan_counts(const uint32_t *__restrict__ counts, int n, int Ns, int chunk_len,
                                                      int bc_chunk_len, const int32_t *__restrict__ slc_start, int32_t *start,
                                                      int32_t *chunk_start, int32_t *part_row_start, int32_t *bc_chunk_start) {
  __shared__ uint32_t part[4][16];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  uint32_t carry[4] = {0u, 0u, 0u, 0u};
  for (int i0 = 0; i0 < n; i0 += 1024) {
    const int i = i0 + tid;
    uint32_t s[4] = {0u, 0u, 0u, 0u}, inc[4];
    if (i < n) {
      const int blk = i % Ns;
      s[0] = counts[i];
      s[1] = (s[0] + chunk_len - 1) / chunk_len;
      s[2] = s[1] * (uint32_t)(slc_start[blk + 1] - slc_start[blk]);
      s[3] = (s[0] + bc_chunk_len - 1) / bc_chunk_len;
    }
#pragma unroll
    for (int x = 0; x < 4; ++x) inc[x] = s[x];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1)
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const uint32_t o = __shfl_up(inc[x], off);
        if (lane >= off) inc[x] += o;
      }
    __syncthreads();  // part may still be read from the previous round
    if (lane == 63)
#pragma unroll
      for (int x = 0; x < 4; ++x) part[x][w] = inc[x];
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      uint32_t base = carry[x], all = 0;
#pragma unroll
      for (int ww = 0; ww < 16; ++ww) {
        const uint32_t p = part[x][ww];
        base += ww < w ? p : 0u;
        all += p;
      }
      inc[x] += base - s[x];
      carry[x] += all;
    }
    if (i < n) {
      start[i] = (int32_t)inc[0]; chunk_start[i] = (int32_t)inc[1]; part_row_start[i] = (int32_t)inc[2]; bc_chunk_start[i] = (int32_t)inc[3];
    }
  }
  if (tid == 0) {
    start[n] = (int32_t)carry[0]; chunk_start[n] = (int32_t)carry[1]; part_row_start[n] = (int32_t)carry[2]; bc_chunk_start[n] = (int32_t)carry[3];
  }
}

// Where the execution order of one chunking is prepared: a chunk's bucket (see m_chunk_order) is counted by the thread
// that places the chunk's first entry.
struct OrderArgs {
  const int32_t *chunk_start;  // [keys+1]
  uint32_t *bins;              // [Hkv * bins_per_head] counters
  int4 *slot;                  // [chunks]: bucket, number inside the bucket, key, chunk inside the key
  ChunkRef *order;             // [chunks] in execution order
  int chunk_len;
};

// Pass 4: every entry to its place: list[start of the key + entries of earlier tiles + entries of the key before it in
// this tile].  R: rounds of 8 entries per thread (POS_TILE * T entries per tile).
template <int R>
__global__ __launch_bounds__(SEL_THREADS) void m_sel_fill(SelArgs a, int n_tiles, const uint32_t *__restrict__ cnt,
                                                          const int32_t *__restrict__ start, int32_t *__restrict__ list,
                                                          uint8_t *__restrict__ rank, OrderArgs o0, OrderArgs o1, int bucket,
                                                          int bins_per_head, bool caller_indices) {
  extern __shared__ __align__(16) uint32_t sel_bits[];
  const int tile = blockIdx.x, g = blockIdx.y, b0 = blockIdx.z * KEY_TILE, nb = min(KEY_TILE, a.Ns - b0);
  for (int i = threadIdx.x; i < nb * TILE_WORDS; i += SEL_THREADS) sel_bits[i] = 0u;
  __syncthreads();
  const int p0 = tile * POS_TILE, npos = min(POS_TILE, a.N - p0);
  // set the bits of all entries of this thread (they stay in registers); an entry whose bit another one owns is dropped
  int b[8 * R];
#pragma unroll
  for (int u = 0; u < 8 * R; ++u) b[u] = sel_block(a, p0, npos, g, u * SEL_THREADS + threadIdx.x);
#pragma unroll
  for (int u = 0; u < 8 * R; ++u) {
    const int pl = (u * SEL_THREADS + (int)threadIdx.x) / a.T;
    const uint32_t bit = 1u << (pl & 31);
    if ((unsigned)(b[u] - b0) >= (unsigned)nb) b[u] = -1;
    else if (atomicOr(&sel_bits[(b[u] - b0) * TILE_WORDS + (pl >> 5)], bit) & bit) b[u] = -1;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 8 * R; ++u) {
    if (b[u] < 0) continue;
    const int e = u * SEL_THREADS + (int)threadIdx.x, pl = e / a.T, j = e - pl * a.T;
    const uint32_t *w = sel_bits + (b[u] - b0) * TILE_WORDS;
    uint32_t before = __popc(w[pl >> 5] & ((1u << (pl & 31)) - 1u));
#pragma unroll
    for (int x = 0; x < TILE_WORDS - 1; ++x) before += x < (pl >> 5) ? __popc(w[x]) : 0u;
    const int key = g * a.Ns + b[u];
    const int r = (int)(cnt[(size_t)key * n_tiles + tile] + before), at = start[key] + r;
    list[at] = caller_indices ? a.perm[p0 + pl] : p0 + pl;
    rank[at] = (uint8_t)j;
    const int bin = g * bins_per_head + (p0 + pl) / bucket;
    auto first = [&](const OrderArgs &o) {
      if (o.order && r % o.chunk_len == 0)
        o.slot[o.chunk_start[key] + r / o.chunk_len] = make_int4(bin, (int)atomicAdd(&o.bins[bin], 1u), key, r / o.chunk_len);
    };
    first(o0);
    first(o1);
  }
}

// Execution order of the work chunks of one chunking: chunks sorted by (KV head, first query position of the chunk), in
// buckets of `bucket` positions.  Chunks that run at the same time then belong to different blocks but to the same stretch
// of tokens, whose query rows they all gather: the rows are fetched into the L2 once instead of once per selected block.
// The order only decides WHEN a chunk runs, never what it computes, so the arbitrary order inside a bucket (the atomic
// counters of m_sel_fill) does not touch any result.  One workgroup per chunking: the prefix of the bucket counters in LDS,
// then every chunk goes to bucket start + number in the bucket.
constexpr int ORDER_BINS = 8192;
__global__ __launch_bounds__(1024) void m_chunk_order(OrderArgs o0, OrderArgs o1, const int32_t *__restrict__ start, int n_keys, int n_bins) {
  __shared__ uint32_t base[ORDER_BINS];
  __shared__ uint32_t part[16];
  const OrderArgs &o = blockIdx.x == 0 ? o0 : o1;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int total = o.chunk_start[n_keys];
  for (int i = tid; i < ORDER_BINS; i += 1024) base[i] = i < n_bins ? o.bins[i] : 0u;
  __syncthreads();
  uint32_t v[ORDER_BINS / 1024], own = 0;
#pragma unroll
  for (int i = 0; i < ORDER_BINS / 1024; ++i) { v[i] = base[tid * (ORDER_BINS / 1024) + i]; own += v[i]; }
  uint32_t inc = own;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t t = __shfl_up(inc, off);
    if (lane >= off) inc += t;
  }
  if (lane == 63) part[w] = inc;
  __syncthreads();
  uint32_t run = inc - own;
  for (int ww = 0; ww < w; ++ww) run += part[ww];
#pragma unroll
  for (int i = 0; i < ORDER_BINS / 1024; ++i) { base[tid * (ORDER_BINS / 1024) + i] = run; run += v[i]; }
  __syncthreads();
  for (int c = tid; c < total; c += 1024) {
    const int4 s = o.slot[c];
    const int first = start[s.z] + s.w * o.chunk_len;
    o.order[base[s.x] + (uint32_t)s.y] = ChunkRef{s.z, s.w, first, min(o.chunk_len, start[s.z + 1] - first)};
  }
}

struct Plan { size_t cnt, counts, start, list, rank, cstart, prow, bcstart, bins, bcslot, slot, bcorder, order, total; };

int pos_tiles(int N) { return (N + POS_TILE - 1) / POS_TILE; }

Plan plan(int N, int Hkv, int T, int Ns) {
  Plan p{};
  size_t off = 0;
  auto take = [&](size_t n) { size_t r = off; off += align_up(n, 256); return r; };
  const size_t keys = (size_t)Hkv * Ns, entries = (size_t)N * Hkv * T;
  p.cnt = take(keys * pos_tiles(N) * 4); p.counts = take(keys * 4 + 4); p.start = take((keys + 1) * 4);
  p.list = take(entries * 4); p.rank = take(entries);
  p.cstart = take((keys + 1) * 4); p.prow = take((keys + 1) * 4); p.bcstart = take((keys + 1) * 4);
  p.bins = take(2 * ORDER_BINS * 4);
  // at most one partly filled chunk per key on top of the full ones
  const size_t bc = entries / BC_CHUNK_MIN + keys + 8, dkv = entries / 256 + keys + 8;
  p.bcslot = take(bc * sizeof(int4)); p.slot = take(dkv * sizeof(int4));
  p.bcorder = take(bc * sizeof(ChunkRef)); p.order = take(dkv * sizeof(ChunkRef));
  p.total = off;
  return p;
}

}  // namespace

size_t sel_index_bytes(int N, int Hkv, int T, int Ns) { return plan(N, Hkv, T, Ns).total; }

SelIndex sel_index_carve(void *ws_, int N, int Hkv, int T, int Ns, int chunk_len, int bc_chunk_len) {
  const Plan p = plan(N, Hkv, T, Ns);
  char *ws = (char *)ws_;
  SelIndex x{};
  x.cnt = (uint32_t *)(ws + p.cnt); x.counts = (uint32_t *)(ws + p.counts); x.start = (int32_t *)(ws + p.start);
  x.list = (int32_t *)(ws + p.list); x.rank = (uint8_t *)(ws + p.rank);
  x.chunk_start = (int32_t *)(ws + p.cstart); x.part_row_start = (int32_t *)(ws + p.prow);
  x.bc_chunk_start = (int32_t *)(ws + p.bcstart); x.bins = (uint32_t *)(ws + p.bins);
  x.bc_slot = (int4 *)(ws + p.bcslot); x.slot = (int4 *)(ws + p.slot);
  x.bc_order = (ChunkRef *)(ws + p.bcorder); x.order = (ChunkRef *)(ws + p.order);
  x.chunk_len = chunk_len; x.bc_chunk_len = bc_chunk_len;
  return x;
}

int sel_index_build(const int32_t *idx, const int32_t *perm, const int32_t *slc_start, int N, int Hkv, int T, int Ns,
                    const SelIndex &x, bool caller_indices, bool want_bc_order, bool want_dkv_order, hipStream_t s) {
  const int tiles = pos_tiles(N), keys = Hkv * Ns;
  // bucket width of the execution orders: Hkv * ceil(N / bucket) buckets fit the LDS table
  int bucket = 64;
  while ((long long)Hkv * ((N + bucket - 1) / bucket) > ORDER_BINS) bucket *= 2;
  const int bph = (N + bucket - 1) / bucket, n_bins = Hkv * bph;
  const SelArgs a{idx, perm, N, Hkv, T, Ns};
  const dim3 grid(tiles, Hkv, (Ns + KEY_TILE - 1) / KEY_TILE);
  const size_t lds = (size_t)(Ns < KEY_TILE ? Ns : KEY_TILE) * TILE_WORDS * 4;
  OrderArgs bc{x.bc_chunk_start, x.bins, x.bc_slot, want_bc_order ? x.bc_order : nullptr, x.bc_chunk_len};
  OrderArgs dkv{x.chunk_start, x.bins + ORDER_BINS, x.slot, want_dkv_order ? x.order : nullptr, x.chunk_len};
  m_sel_count<<<grid, SEL_THREADS, lds, s>>>(a, tiles, x.cnt, x.bins, ORDER_BINS, n_bins);
  m_sel_scan_tiles<<<(keys + 3) / 4, 256, 0, s>>>(x.cnt, keys, tiles, x.counts);
  m_scan_counts<<<1, 1024, 0, s>>>(x.counts, keys, Ns, x.chunk_len, x.bc_chunk_len, slc_start, x.start, x.chunk_start,
                                   x.part_row_start, x.bc_chunk_start);
  if (T <= 16) m_sel_fill<1><<<grid, SEL_THREADS, lds, s>>>(a, tiles, x.cnt, x.start, x.list, x.rank, bc, dkv, bucket, bph, caller_indices);
  else if (T <= 32) m_sel_fill<2><<<grid, SEL_THREADS, lds, s>>>(a, tiles, x.cnt, x.start, x.list, x.rank, bc, dkv, bucket, bph, caller_indices);
  else m_sel_fill<4><<<grid, SEL_THREADS, lds, s>>>(a, tiles, x.cnt, x.start, x.list, x.rank, bc, dkv, bucket, bph, caller_indices);
  if (want_bc_order && want_dkv_order) m_chunk_order<<<2, 1024, 0, s>>>(bc, dkv, x.start, keys, n_bins);
  else if (want_bc_order) m_chunk_order<<<1, 1024, 0, s>>>(bc, bc, x.start, keys, n_bins);
  else if (want_dkv_order) m_chunk_order<<<1, 1024, 0, s>>>(dkv, dkv, x.start, keys, n_bins);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}
