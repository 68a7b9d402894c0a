// Inverse of the selection (gfx950): for every (KV head, selection block) the ascending list of sorted positions of the
// query tokens whose row of the index tensor I (Algorithm 1) holds the block, each with its rank in that row, and the cuts
// of every list into work chunks.  The block-centric selection kernels (forward and dQ) and the key-centric dK/dV kernel
// walk these lists.  A counting sort over tiles of POS_TILE sorted positions: a tile's selections are marked in a bit
// matrix in LDS (integer OR: order independent), so that the population count below a bit is the entry's rank inside its
// tile; per-tile counts are turned into offsets, and every entry then writes itself to its final place.  Integer work
// only, and the lists do not depend on scheduling.
// Bound: latency of two to five small dependent launches (every pass reads or writes a few MB), so a tile is small enough that all
// its loads are in flight at once, and in small problems the prefix sums are the work of whichever workgroup of the first pass ends last.
// Kernel times: 11k tokens, top-8, 226 lists: 22 us in two launches (25 us in five); 2k tokens, 66 lists: 18 us (28); 62k tokens,
// top-16, 994 lists: 60 us in five.
#include "mfma_launch.h"
#include "sel_order.h"

#include <mutex>

namespace {

constexpr int POS_TILE = 256;              // sorted positions per tile (8 words of 32 bits per key)
constexpr int TILE_WORDS = POS_TILE / 32;
constexpr int KEY_TILE = 2048;             // selection blocks of one KV head a workgroup covers: 64 KB of bits
constexpr int SEL_THREADS = 512;
constexpr int FUSED_COUNTS = 16384;  // see sel_index_build
constexpr int ORDER_STEP = 64;  // keys per class of block lengths

struct SelArgs {
  const int32_t *idx, *perm;
  int N, Hkv, T, Ns;
};

__device__ inline int sel_block(const SelArgs &a, int p0, int npos, int g, int e) {  // block of entry e of the tile, or -1
  const int pl = e / a.T, j = e - pl * a.T;
  return pl < npos ? a.idx[((size_t)a.perm[p0 + pl] * a.Hkv + g) * a.T + j] : -1;
}

// A store that other workgroups' loads find once it is complete (written through at device scope).
__device__ inline void store_shared(uint32_t *p, uint32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Whether the calling workgroup is the last of `total` to get here; what the others wrote before with store_shared is then there for
// it to read.  (Every thread waits for its own stores to be complete before the workgroup draws its ticket.  A release fence would
// write the whole L2 back, once per wavefront or workgroup: 160 us for the 12 of this pass at 21k tokens.)
__device__ inline bool last_workgroup(uint32_t *ticket, uint32_t total) {
  __shared__ bool last;
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  __syncthreads();
  if (threadIdx.x == 0) last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == total - 1u;
  __syncthreads();
  if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  return last;
}

struct ScanArgs {
  uint32_t *counts;            // [n] entries per key
  const int32_t *slc_start;
  int32_t *start, *chunk_start, *part_row_start, *bc_chunk_start;  // [n + 1] each
  int n, Ns, chunk_len, bc_chunk_len;
};

// From the per-(g, block) selector counts, four exclusive prefix sums over the n keys by one workgroup of NT threads:
// start (list offsets), chunk_start (work chunks of chunk_len query tokens), part_row_start (rows of partial sums:
// chunks x keys of the block), bc_chunk_start (work chunks of bc_chunk_len query tokens).
template <int NT>
__device__ inline void scan_counts(const ScanArgs &a) {
  constexpr int NW = NT / 64;
  __shared__ uint32_t part[4][NW];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  uint32_t carry[4] = {0u, 0u, 0u, 0u};
  for (int i0 = 0; i0 < a.n; i0 += NT) {
    const int i = i0 + tid;
    uint32_t s[4] = {0u, 0u, 0u, 0u}, inc[4];
    if (i < a.n) {
      const int blk = i % a.Ns;
      s[0] = a.counts[i];
      s[1] = (s[0] + a.chunk_len - 1) / a.chunk_len;
      s[2] = s[1] * (uint32_t)(a.slc_start[blk + 1] - a.slc_start[blk]);
      s[3] = (s[0] + a.bc_chunk_len - 1) / a.bc_chunk_len;
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
      for (int ww = 0; ww < NW; ++ww) {
        const uint32_t p = part[x][ww];
        base += ww < w ? p : 0u;
        all += p;
      }
      inc[x] += base - s[x];
      carry[x] += all;
    }
    if (i < a.n) {
      a.start[i] = (int32_t)inc[0]; a.chunk_start[i] = (int32_t)inc[1]; a.part_row_start[i] = (int32_t)inc[2]; a.bc_chunk_start[i] = (int32_t)inc[3];
    }
  }
  if (tid == 0) {
    a.start[a.n] = (int32_t)carry[0]; a.chunk_start[a.n] = (int32_t)carry[1]; a.part_row_start[a.n] = (int32_t)carry[2]; a.bc_chunk_start[a.n] = (int32_t)carry[3];
  }
}

// Where the chunks of every key begin in an order by falling block length (both chunkings), by one workgroup: the longest work comes
// first, so that what ends last is short.  A counting sort over lengths in steps of 8 keys; the order inside a step is arbitrary
// (it decides when a chunk runs, never what it computes).
template <int NT>
__device__ inline void order_by_length(const ScanArgs &a, int32_t *base, int32_t *bc_base) {
  constexpr int STEPS = 64;
  __shared__ uint32_t at[2][STEPS];  // chunks per step, then where the next key's go
  for (int i = threadIdx.x; i < 2 * STEPS; i += NT) at[i / STEPS][i % STEPS] = 0u;
  __syncthreads();
  auto step_of = [&](int i) { return STEPS - 1 - min((a.slc_start[i % a.Ns + 1] - a.slc_start[i % a.Ns]) / 8, STEPS - 1); };
  auto place = [&](int i, int s, uint32_t &x, uint32_t &y) {
    const uint32_t c = a.counts[i];
    x = atomicAdd(&at[0][s], (c + a.chunk_len - 1) / a.chunk_len);
    y = atomicAdd(&at[1][s], (c + a.bc_chunk_len - 1) / a.bc_chunk_len);
  };
  uint32_t x, y;
  for (int i = threadIdx.x; i < a.n; i += NT) place(i, step_of(i), x, y);
  __syncthreads();
  if (threadIdx.x < 2 * STEPS) {  // (a wavefront per chunking)
    const int w = threadIdx.x / STEPS, lane = threadIdx.x % STEPS;
    const uint32_t own = at[w][lane];
    uint32_t inc = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t o = __shfl_up(inc, off);
      if (lane >= off) inc += o;
    }
    at[w][lane] = inc - own;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < a.n; i += NT) {
    place(i, step_of(i), x, y);
    base[i] = (int32_t)x;
    bc_base[i] = (int32_t)y;
  }
}

// Pass 1: entries per (key, tile).  cnt[key][stride].  Workgroup column (., 0, 0) also clears the counters of the last pass.  With
// a ticket (a word that is 0 when the kernel starts) the last workgroup goes on with passes 2 and 3, a thread per key.
__global__ __launch_bounds__(SEL_THREADS) void m_sel_count(SelArgs a, int n_tiles, int stride, uint32_t *__restrict__ cnt,
                                                           uint32_t *__restrict__ bins, int bins_stride, int n_bins, uint32_t *ticket,
                                                           ScanArgs sc, int32_t *base, int32_t *bc_base) {
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
    const uint32_t count = __popc(x.x) + __popc(x.y) + __popc(x.z) + __popc(x.w) + __popc(y.x) + __popc(y.y) + __popc(y.z) + __popc(y.w);
    uint32_t *to = &cnt[((size_t)g * a.Ns + b0 + i) * stride + tile];
    if (ticket) store_shared(to, count);
    else *to = count;  // (to the next kernel; written through 60k tokens' counts take 40 us for 27)
  }
  if (!ticket || !last_workgroup(ticket, gridDim.x * gridDim.y * gridDim.z)) return;
  for (int key = threadIdx.x; key < sc.n; key += SEL_THREADS) {
    uint4 *row = reinterpret_cast<uint4 *>(cnt + (size_t)key * stride);
    const int n4 = stride / 4;
    uint32_t run = 0;
    for (int t0 = 0; t0 < n4; t0 += 8) {  // (32 counts in flight, under no condition; what lies behind the last tile is not counted)
      uint4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = row[min(t0 + u, n4 - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        uint32_t c[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t own = 4 * (t0 + u) + j < n_tiles ? c[j] : 0u;
          c[j] = run;
          run += own;
        }
        if (t0 + u < n4) row[t0 + u] = make_uint4(c[0], c[1], c[2], c[3]);
      }
    }
    sc.counts[key] = run;
  }
  __syncthreads();
  scan_counts<SEL_THREADS>(sc);
  if (base) order_by_length<SEL_THREADS>(sc, base, bc_base);
}

// Pass 2: per key (one wavefront each) the exclusive prefix of its counts over the tiles, in place, and their sum.
__global__ __launch_bounds__(256) void m_sel_scan_tiles(uint32_t *__restrict__ cnt, int n_keys, int n_tiles, int stride, uint32_t *__restrict__ counts) {
  const int key = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (key >= n_keys) return;
  uint32_t *row = cnt + (size_t)key * stride;
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

// Pass 3, one workgroup: the prefix sums over the keys.  (By the workgroup of pass 2 that ends last, of 256 threads, instead: 62k tokens,
// 1300 lists 14 us for 5 + 6 in two launches; 24k tokens, 4200 lists 44 for 5 + 14; 60k, 8200 lists 62 for 7 + 24.)
__global__ __launch_bounds__(1024) void m_sel_scan_keys(ScanArgs sc, int32_t *base, int32_t *bc_base) {
  scan_counts<1024>(sc);
  if (base) order_by_length<1024>(sc, base, bc_base);
}

// Where the execution order of one chunking is prepared: a chunk's bucket (see m_chunk_order) is counted by the thread
// that places the chunk's first entry.
struct OrderArgs {
  const int32_t *chunk_start;  // [keys+1]
  uint32_t *bins;              // [Hkv * bins_per_head] counters
  int4 *slot;                  // [chunks]: bucket, number inside the bucket, key, chunk inside the key
  ChunkRef *order;             // [chunks] in execution order
  int chunk_len;
  const int32_t *base;         // [keys] first place of every key's chunks, which m_sel_fill then writes itself; or null: m_chunk_order
};

// Pass 4: every entry to its place: list[start of the key + entries of earlier tiles + entries of the key before it in
// this tile].  R: rounds of 8 entries per thread (POS_TILE * T entries per tile).
template <int R>
__global__ __launch_bounds__(SEL_THREADS) void m_sel_fill(SelArgs a, int n_tiles, int stride, const uint32_t *__restrict__ cnt,
                                                          const int32_t *__restrict__ start, int32_t *__restrict__ list,
                                                          uint8_t *__restrict__ rank, OrderArgs o0, OrderArgs o1, const int32_t *__restrict__ slc_start,
                                                          SelOrder ord, bool caller_indices) {
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
    const int r = (int)(cnt[(size_t)key * stride + tile] + before), at = start[key] + r;
    list[at] = caller_indices ? a.perm[p0 + pl] : p0 + pl;
    rank[at] = (uint8_t)j;
    auto first = [&](const OrderArgs &o) {
      if (!o.order || r % o.chunk_len != 0) return;
      const int c = r / o.chunk_len;
      if (o.base) o.order[o.base[key] + c] = ChunkRef{key, c, at, min(o.chunk_len, start[key + 1] - at)};
      else {
        const int cls = ord.classes - 1 - min((slc_start[b[u] + 1] - slc_start[b[u]]) / ORDER_STEP, ord.classes - 1);
        const int bin = (cls * a.Hkv + g) * ord.per_head + (p0 + pl) / ord.bucket;
        o.slot[o.chunk_start[key] + c] = make_int4(bin, (int)atomicAdd(&o.bins[bin], 1u), key, c);
      }
    };
    first(o0);
    first(o1);
  }
}

// Execution order of the work chunks of one chunking: chunks sorted by (class of block lengths, falling; KV head; first query
// position of the chunk, in buckets of `bucket` positions).  The longest work comes first, so that what ends last is short; inside a
// class chunks that run at the same time belong to different blocks but to the same stretch
// of tokens, whose query rows they all gather: the rows are fetched once instead of once per selected block.
// m_slc_fwd_bc / m_slc_bwd, us, by stretches alone (a contiguous run per XCD in the forward kernel), by falling length alone, and as
// here: 62k tokens 928 / 3457, 923 / 3236, 887 / 3012; 147k in four shapes 2636 / 7397, 2196 / 7218, 2073 / 7036; sequences, whose
// blocks are all of one length, 678 / 1334, 669 / 1429, 613 / 1343; 153k, heads of 128, forward 9.8, 9.6, 9.2 ms.
// The order only decides WHEN a chunk runs, never what it computes, so the arbitrary order inside a bucket (the atomic
// counters of m_sel_fill) does not touch any result.  One workgroup per chunking: the prefix of the bucket counters in LDS,
// then every chunk goes to bucket start + number in the bucket.
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

struct Plan { size_t cnt, counts, base, start, list, rank, cstart, prow, bcstart, bins, bcslot, slot, bcorder, order, total; };

int pos_tiles(int N) { return (N + POS_TILE - 1) / POS_TILE; }
int tile_stride(int N) { return (pos_tiles(N) + 3) / 4 * 4; }  // rows of the per-tile counts start on 16 bytes

Plan plan(int N, int Hkv, int T, int Ns) {
  Plan p{};
  size_t off = 0;
  auto take = [&](size_t n) { size_t r = off; off += align_up(n, 256); return r; };
  const size_t keys = (size_t)Hkv * Ns, entries = (size_t)N * Hkv * T;
  p.cnt = take(keys * tile_stride(N) * 4); p.counts = take(keys * 4 + 4); p.base = take(2 * keys * 4); p.start = take((keys + 1) * 4);
  p.list = take(entries * 4); p.rank = take(entries);
  p.cstart = take((keys + 1) * 4); p.prow = take((keys + 1) * 4); p.bcstart = take((keys + 1) * 4);
  p.bins = take(2 * ORDER_BINS * 4 + 4);
  // at most one partly filled chunk per key on top of the full ones
  const size_t bc = entries / BC_CHUNK_MIN + keys + 8, dkv = entries / DKV_CHUNK_MIN + keys + 8;
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
  x.bc_chunk_start = (int32_t *)(ws + p.bcstart); x.bins = (uint32_t *)(ws + p.bins); x.ticket = x.bins + 2 * ORDER_BINS;
  x.base = (int32_t *)(ws + p.base);
  x.by_length = sel_order(N, Hkv).by_length;
  x.bc_slot = (int4 *)(ws + p.bcslot); x.slot = (int4 *)(ws + p.slot);
  x.bc_order = (ChunkRef *)(ws + p.bcorder); x.order = (ChunkRef *)(ws + p.order);
  x.chunk_len = chunk_len; x.bc_chunk_len = bc_chunk_len;
  return x;
}

int sel_index_build(const int32_t *idx, const int32_t *perm, const int32_t *slc_start, int N, int Hkv, int T, int Ns,
                    const SelIndex &x, bool caller_indices, bool want_bc_order, bool want_dkv_order, hipStream_t s) {
  const int tiles = pos_tiles(N), stride = tile_stride(N), keys = Hkv * Ns;
  // The last workgroup of the first pass does the second and third as well where the counts are few (a thread per key).
  const bool fused = (long long)keys * stride <= FUSED_COUNTS;
  int32_t *const base = x.by_length ? x.base : nullptr, *const bc_base = x.by_length ? x.base + keys : nullptr;
  const SelOrder ord = sel_order(N, Hkv);
  const int n_bins = x.by_length ? 0 : ord.classes * Hkv * ord.per_head;
  const SelArgs a{idx, perm, N, Hkv, T, Ns};
  const dim3 grid(tiles, Hkv, (Ns + KEY_TILE - 1) / KEY_TILE);
  const size_t lds = (size_t)(Ns < KEY_TILE ? Ns : KEY_TILE) * TILE_WORDS * 4;
  const ScanArgs sc{x.counts, slc_start, x.start, x.chunk_start, x.part_row_start, x.bc_chunk_start, keys, Ns, x.chunk_len, x.bc_chunk_len};
  OrderArgs bc{x.bc_chunk_start, x.bins, x.bc_slot, want_bc_order ? x.bc_order : nullptr, x.bc_chunk_len, bc_base};
  OrderArgs dkv{x.chunk_start, x.bins + ORDER_BINS, x.slot, want_dkv_order ? x.order : nullptr, x.chunk_len, base};
  static std::once_flag once;  // its own LDS stands beside up to 64 KB of bits
  std::call_once(once, [] { (void)hipFuncSetAttribute((const void *)m_sel_count, hipFuncAttributeMaxDynamicSharedMemorySize, KEY_TILE * TILE_WORDS * 4); });
  m_sel_count<<<grid, SEL_THREADS, lds, s>>>(a, tiles, stride, x.cnt, x.bins, ORDER_BINS, n_bins, fused ? x.ticket : nullptr, sc, base, bc_base);
  if (!fused) {
    m_sel_scan_tiles<<<(keys + 3) / 4, 256, 0, s>>>(x.cnt, keys, tiles, stride, x.counts);
    m_sel_scan_keys<<<1, 1024, 0, s>>>(sc, base, bc_base);
  }
  if (T <= 16) m_sel_fill<1><<<grid, SEL_THREADS, lds, s>>>(a, tiles, stride, x.cnt, x.start, x.list, x.rank, bc, dkv, slc_start, ord, caller_indices);
  else if (T <= 32) m_sel_fill<2><<<grid, SEL_THREADS, lds, s>>>(a, tiles, stride, x.cnt, x.start, x.list, x.rank, bc, dkv, slc_start, ord, caller_indices);
  else m_sel_fill<4><<<grid, SEL_THREADS, lds, s>>>(a, tiles, stride, x.cnt, x.start, x.list, x.rank, bc, dkv, slc_start, ord, caller_indices);
  if (x.by_length) return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
  if (want_bc_order && want_dkv_order) m_chunk_order<<<2, 1024, 0, s>>>(bc, dkv, x.start, keys, n_bins);
  else if (want_bc_order) m_chunk_order<<<1, 1024, 0, s>>>(bc, bc, x.start, keys, n_bins);
  else if (want_dkv_order) m_chunk_order<<<1, 1024, 0, s>>>(dkv, dkv, x.start, keys, n_bins);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}
