// Inverse of the selection (gfx950): for every (KV head, selection block) the ascending list of sorted positions of the
// query tokens whose row of the index tensor I (Algorithm 1) holds the block, each with its rank in that row, and the cuts
// of every list into work chunks.  The block-centric selection kernels (forward and dQ) and the key-centric dK/dV kernel
// walk these lists.  A counting sort over tiles of POS_TILE sorted positions: a tile's selections are marked in a bit
// matrix in LDS (integer OR: order independent), so that the population count below a bit is the entry's rank inside its
// tile; per-tile counts are turned into offsets, and every entry then writes itself to its final place.  Integer work
// only, and the lists do not depend on scheduling.
// Bound: latency of one to five small dependent launches (every pass reads or writes a few MB), so a tile is small enough that all
// its loads are in flight at once, and in small problems the prefix sums are the work of whichever workgroup of the first pass ends last, or
// the counts come with the selection itself (sel_counted).
// Kernel times: 11k tokens, top-8, 226 lists: 22 us in two launches (25 us in five), 12 in one; 2k tokens, 66 lists: 18 us (28), 10;
// 62k tokens, top-16, 994 lists: 60 us in five.
#include "cmp_form.h"
#include "sel_device.h"

#include <mutex>

namespace {

constexpr int KEY_TILE = 2048;             // selection blocks of one KV head a workgroup covers: 64 KB of bits
constexpr int SEL_THREADS = 512;
constexpr int FUSED_COUNTS = 16384;  // see sel_index_job

__global__ __launch_bounds__(SEL_THREADS) void m_sel_count(SelJob j) {
  extern __shared__ __align__(16) uint32_t sel_bits[];
  sel_count<SEL_THREADS>(j, SelPlace{(int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z * j.key_tile}, sel_bits);
}
template <int R>
__global__ __launch_bounds__(SEL_THREADS) void m_sel_fill(SelJob j) {
  extern __shared__ __align__(16) uint32_t sel_bits[];
  const SelPlace at{(int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z * j.key_tile};
  sel_fill<SEL_THREADS, R>(j, at, sel_bits, [&] { return sel_scanned(j, at); });
}

// Exclusive prefix over the workgroup's threads, and the sum; part: SEL_THREADS / 64 words of LDS of the call's own.
__device__ inline uint32_t prefix_over_threads(uint32_t own, uint32_t *part, uint32_t *sum) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t inc = own;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t o = __shfl_up(inc, off);
    if (lane >= off) inc += o;
  }
  if (lane == 63) part[w] = inc;
  __syncthreads();
  uint32_t base = 0, all = 0;
#pragma unroll
  for (int ww = 0; ww < SEL_THREADS / 64; ++ww) {
    base += ww < w ? part[ww] : 0u;
    all += part[ww];
  }
  *sum = all;
  return base + inc - own;
}

// The whole index in one launch, where the compression kernel has left the counts as [tile][key] (sel_counted): every workgroup forms
// the prefix sums it needs, a thread per key, while its entries are on their way, and fills its tile.
template <int R>
__global__ __launch_bounds__(SEL_THREADS) void m_sel_fill_counted(SelJob j) {
  extern __shared__ __align__(16) uint32_t sel_bits[];
  constexpr int NW = SEL_THREADS / 64, STEPS = 64;
  __shared__ uint32_t part[2][NW], steps[NW][STEPS], before[SEL_THREADS];
  __shared__ int32_t start[SEL_THREADS + 1], base[SEL_THREADS];
  const SelPlace at{(int)blockIdx.x, (int)blockIdx.y, 0};
  sel_fill<SEL_THREADS, R>(j, at, sel_bits, [&] {
    const int key = threadIdx.x, lane = key & 63, w = key >> 6, n = j.sc.n, own_key = min(key, n - 1), blk = own_key % j.a.Ns;
    const int len = j.sc.slc_start[blk + 1] - j.sc.slc_start[blk];
    uint32_t all = 0, earlier = 0;
    for (int t0 = 0; t0 < j.tiles; t0 += 16) {  // (16 counts in flight, under no condition)
      uint32_t v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = j.cnt[(size_t)min(t0 + u, j.tiles - 1) * n + own_key];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        all += t0 + u < j.tiles ? v[u] : 0u;
        earlier += t0 + u < at.tile ? v[u] : 0u;
      }
    }
    if (key >= n) all = 0u;
    for (int i = lane; i < STEPS; i += 64) steps[w][i] = 0u;
    uint32_t entries, chunks;
    start[key] = (int32_t)prefix_over_threads(all, part[0], &entries);
    before[key] = earlier;
    if (key == n - 1) start[n] = (int32_t)entries;
    // the places of the chunks by falling block length, as order_by_length has them, but the same in every workgroup: inside a step of
    // 8 keys by key
    const uint32_t c = (all + j.sc.bc_chunk_len - 1) / j.sc.bc_chunk_len;
    const int step = STEPS - 1 - min(len / 8, STEPS - 1);
    if (c) atomicAdd(&steps[w][step], c);
    uint64_t same = ~0ull;  // lanes of this step
#pragma unroll
    for (int bit = 0; bit < 6; ++bit) {
      const uint64_t m = __ballot(step >> bit & 1);
      same &= step >> bit & 1 ? m : ~m;
    }
    same &= (1ull << lane) - 1ull;
    uint32_t mine = 0;  // chunks of the keys before this one in the same step and wavefront
    for (int bit = 0; __any(c >> bit); ++bit) mine += (uint32_t)__popcll(__ballot(c >> bit & 1u) & same) << bit;
    __syncthreads();
    uint32_t of_step = 0;  // (the first wavefront: a thread per step)
    if (key < STEPS)
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) of_step += steps[ww][key];
    uint32_t run = prefix_over_threads(of_step, part[1], &chunks);
    if (key < STEPS)
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) {
        const uint32_t x = steps[ww][key];
        steps[ww][key] = run;
        run += x;
      }
    __syncthreads();
    base[key] = (int32_t)(steps[w][step] + mine);
    if (blockIdx.x == 0 && blockIdx.y == 0 && key == 0) j.sc.bc_chunk_start[n] = (int32_t)chunks;
    __syncthreads();
    return SelKeys{start, before, 1, base, nullptr};
  });
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

SelJob sel_index_job(const int32_t *idx, const int32_t *perm, const int32_t *slc_start, int N, int Hkv, int T, int Ns, const SelIndex &x,
                     bool caller_indices, bool want_bc_order, bool want_dkv_order, bool beside) {
  SelJob j{};
  const int keys = Hkv * Ns;
  j.a = SelArgs{idx, perm, N, Hkv, T, Ns};
  j.tiles = pos_tiles(N); j.stride = tile_stride(N); j.key_tile = beside ? SEL_BESIDE_KEYS : KEY_TILE;
  j.cnt = x.cnt; j.bins = x.bins; j.bins_stride = ORDER_BINS;
  // The last workgroup of the first pass does the second and third as well where the counts are few (a thread per key).
  j.ticket = (long long)keys * j.stride <= FUSED_COUNTS ? x.ticket : nullptr;
  j.base = x.by_length ? x.base : nullptr; j.bc_base = x.by_length ? x.base + keys : nullptr;
  j.ord = sel_order(N, Hkv);
  j.n_bins = x.by_length ? 0 : j.ord.classes * Hkv * j.ord.per_head;
  j.sc = ScanArgs{x.counts, slc_start, x.start, x.chunk_start, x.part_row_start, x.bc_chunk_start, keys, Ns, x.chunk_len, x.bc_chunk_len};
  j.bc = OrderArgs{x.bc_chunk_start, x.bins, x.bc_slot, want_bc_order ? x.bc_order : nullptr, x.bc_chunk_len, j.bc_base};
  j.dkv = OrderArgs{x.chunk_start, x.bins + ORDER_BINS, x.slot, want_dkv_order ? x.order : nullptr, x.chunk_len, j.base};
  j.list = x.list; j.rank = x.rank; j.caller_indices = caller_indices;
  return j;
}

int sel_index_count(const SelJob &j, hipStream_t s) {
  static std::once_flag once;  // its own LDS stands beside up to 64 KB of bits
  std::call_once(once, [] { (void)hipFuncSetAttribute((const void *)m_sel_count, hipFuncAttributeMaxDynamicSharedMemorySize, KEY_TILE * TILE_WORDS * 4); });
  m_sel_count<<<dim3(j.tiles, j.a.Hkv, j.parts()), SEL_THREADS, j.lds_bytes(), s>>>(j);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}
int sel_index_scan(const SelJob &j, hipStream_t s) {
  if (j.ticket) return SSA_OK;  // (done)
  m_sel_scan_tiles<<<(j.sc.n + 3) / 4, 256, 0, s>>>(j.cnt, j.sc.n, j.tiles, j.stride, j.sc.counts);
  m_sel_scan_keys<<<1, 1024, 0, s>>>(j.sc, j.base, j.bc_base);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}
int sel_index_fill(const SelJob &j, hipStream_t s) {
  const dim3 n(j.tiles, j.a.Hkv, j.parts());
  if (j.a.T <= 16) m_sel_fill<1><<<n, SEL_THREADS, j.lds_bytes(), s>>>(j);
  else if (j.a.T <= 32) m_sel_fill<2><<<n, SEL_THREADS, j.lds_bytes(), s>>>(j);
  else m_sel_fill<4><<<n, SEL_THREADS, j.lds_bytes(), s>>>(j);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}
int sel_index_order(const SelJob &j, hipStream_t s) {
  if (j.base) return SSA_OK;  // (by length: written by the fill pass)
  const OrderArgs &bc = j.bc.order ? j.bc : j.dkv, &dkv = j.dkv.order ? j.dkv : j.bc;
  if (bc.order) m_chunk_order<<<j.bc.order && j.dkv.order ? 2 : 1, 1024, 0, s>>>(bc, dkv, j.sc.start, j.sc.n, j.n_bins);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}

// A thread per list, and few enough counts that every workgroup reads all of them.  The compression kernel takes as long as before, 3 us more
// at 11k tokens.  Whole forward, counted apart / by it: 2k tokens, 32 heads of 32 79.5 / 72.4 us, 11k, 16 heads of 64 294.8 / 286.4, a
// layer of 5.5k 209.8 / 203.3.
bool sel_counted(int D, int hs, int s_max, int N, int Hkv, int Ns) {
  const long long keys = (long long)Hkv * Ns;
  return keys <= SEL_THREADS && keys * pos_tiles(N) <= FUSED_COUNTS && sel_order(N, Hkv).by_length && cmp_counts(D, hs, s_max, Ns);
}

int sel_index_build(const int32_t *idx, const int32_t *perm, const int32_t *slc_start, int N, int Hkv, int T, int Ns,
                    const SelIndex &x, bool caller_indices, bool want_bc_order, bool want_dkv_order, bool counted, hipStream_t s) {
  const SelJob j = sel_index_job(idx, perm, slc_start, N, Hkv, T, Ns, x, caller_indices, want_bc_order, want_dkv_order, false);
  if (counted) {
    const dim3 n(j.tiles, Hkv);
    if (T <= 16) m_sel_fill_counted<1><<<n, SEL_THREADS, j.lds_bytes(), s>>>(j);
    else if (T <= 32) m_sel_fill_counted<2><<<n, SEL_THREADS, j.lds_bytes(), s>>>(j);
    else m_sel_fill_counted<4><<<n, SEL_THREADS, j.lds_bytes(), s>>>(j);
    return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
  }
  int rc = sel_index_count(j, s);
  if (rc == SSA_OK) rc = sel_index_scan(j, s);
  if (rc == SSA_OK) rc = sel_index_fill(j, s);
  if (rc == SSA_OK) rc = sel_index_order(j, s);
  return rc;
}
