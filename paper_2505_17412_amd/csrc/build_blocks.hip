// Block partition, token sort and block start arrays for SSA on gfx950.
//
// Paper, Sec. "Spatial Sparse Attention": tokens whose voxels fall into the same m^3 sub-grid form a block;
// tokens are sorted by block and the first-token index of every block (array C of Algorithm 1) is kept.
// Here one Morton-order sort serves the three block granularities (all sides are powers of two, so every
// aligned cube is a contiguous run of the Morton order): key = (batch item << 3*bits) | Morton(x,y,z).
// Integer work only; results are bit-exact and independent of scheduling (stable LSD radix sort, no
// order-dependent atomics).
//
// Bound: launch latency (62k tokens are 0.7 MB in, 3 MB out: a microsecond of memory time), so the work is cut into as few
// dependent launches as possible: 11-bit digits (two passes up to 22 key bits instead of three), the key kernel counts the
// first digit, every scatter workgroup forms its own offsets from the tile histograms (about 32 tiles below 256k tokens, a
// tile taking 1..16 keys per thread), the last scatter writes straight into the handle, and the kernel that finds the
// maxima hands the counts to the host through pinned memory.  Seven launches instead of 18 plus four copies; with the
// allocations kept (see DevicePool), a build of 62k tokens, its arrays read out and destroyed: 228 -> 112 us (two thirds of it on the host).
#include "ssa_internal.h"
#include "device_pool.h"

#include <mutex>
#include <vector>

namespace {

constexpr int SORT_THREADS = 512, SORT_WAVES = SORT_THREADS / 64;
constexpr int DIGIT_BITS_MAX = 11, BINS_MAX = 1 << DIGIT_BITS_MAX;

enum { META_ERR = 0, META_NC, META_NS, META_NW, META_SMAX, META_CMAX, META_SLC_TOK, META_WIN_TOK, META_CMP_TOK, META_SLC_128,
       META_SLC_256, META_N, META_DONE = META_N, META_INTS };

// Spread the low 10 bits of v so that bit i lands on bit 3i.
__device__ inline uint32_t spread3(uint32_t v) {
  v &= 0x3FFu;
  v = (v | (v << 16)) & 0x030000FFu;
  v = (v | (v << 8)) & 0x0300F00Fu;
  v = (v | (v << 4)) & 0x030C30C3u;
  v = (v | (v << 2)) & 0x09249249u;
  return v;
}

// A tile is SORT_THREADS * R consecutive keys; wavefront w of its workgroup owns keys 64*R*w .., R rounds of 64.
template <int R>
__device__ inline int tile_key(int round) {
  return blockIdx.x * (SORT_THREADS * R) + (threadIdx.x >> 6) * (64 * R) + round * 64 + (threadIdx.x & 63);
}

// Keys of all tokens and the tile histograms of the first digit (hist[tile][digit]).  err[tile]: bit 0 bad batch offsets,
// bit 1 a coordinate out of range.  Workgroup 0 clears the maxima.
template <int R>
__global__ __launch_bounds__(SORT_THREADS) void k_keys_hist(const int32_t *__restrict__ coords, const int32_t *__restrict__ offs,
                                                            int N, int B, int G, int bits, int dbits, uint64_t *__restrict__ keys,
                                                            uint32_t *__restrict__ hist, int32_t *__restrict__ err, int32_t *meta) {
  __shared__ uint32_t h[BINS_MAX];
  __shared__ int bad_any;
  const int nb = 1 << dbits;
  for (int i = threadIdx.x; i < nb; i += SORT_THREADS) h[i] = 0;
  if (threadIdx.x == 0) bad_any = 0;
  if (blockIdx.x == 0 && threadIdx.x < META_INTS) meta[threadIdx.x] = 0;
  __syncthreads();
  int bad_bits = 0;
  for (int j = blockIdx.x * SORT_THREADS + threadIdx.x; j <= B; j += gridDim.x * SORT_THREADS) {
    const int o = offs[j];
    if ((j == 0 && o != 0) || (j == B && o != N) || (j > 0 && o < offs[j - 1]) || o < 0 || o > N) bad_bits |= 1;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = tile_key<R>(r);
    if (i >= N) continue;
    int lo = 0, hi = B;  // offs[lo] <= i < offs[hi] for valid offsets
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (offs[mid] <= i) lo = mid; else hi = mid;
    }
    int x = coords[3 * i], y = coords[3 * i + 1], z = coords[3 * i + 2];
    if ((unsigned)x >= (unsigned)G || (unsigned)y >= (unsigned)G || (unsigned)z >= (unsigned)G) {
      bad_bits |= 2;
      x = y = z = 0;
    }
    const uint64_t code = (uint64_t)((spread3((uint32_t)x) << 2) | (spread3((uint32_t)y) << 1) | spread3((uint32_t)z));
    const uint64_t key = ((uint64_t)lo << (3 * bits)) | code;
    keys[i] = key;
    atomicAdd(&h[(uint32_t)key & (uint32_t)(nb - 1)], 1u);
  }
  if (bad_bits) atomicOr(&bad_any, bad_bits);
  __syncthreads();
  for (int i = threadIdx.x; i < nb; i += SORT_THREADS) hist[(size_t)blockIdx.x * nb + i] = h[i];
  if (threadIdx.x == 0) err[blockIdx.x] = bad_any;
}

// Tile histograms of a later digit.
template <int R>
__global__ __launch_bounds__(SORT_THREADS) void k_sort_hist(const uint64_t *__restrict__ keys, int N, int shift, int dbits,
                                                            uint32_t *__restrict__ hist) {
  __shared__ uint32_t h[BINS_MAX];
  const int nb = 1 << dbits;
  for (int i = threadIdx.x; i < nb; i += SORT_THREADS) h[i] = 0;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = tile_key<R>(r);
    if (i < N) atomicAdd(&h[(uint32_t)(keys[i] >> shift) & (uint32_t)(nb - 1)], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nb; i += SORT_THREADS) hist[(size_t)blockIdx.x * nb + i] = h[i];
}

// Exclusive prefix sum over the `n` threads of a workgroup (n <= 1024 a multiple of 64): returns the sum of v over the
// threads before this one; *total (optional) receives the sum over all threads.  `part` holds n/64 + 1 words of LDS.
__device__ inline uint32_t block_exclusive_scan(uint32_t v, uint32_t *part, uint32_t *total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  uint32_t inc = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t t = __shfl_up(inc, off);
    if (lane >= off) inc += t;
  }
  __syncthreads();  // part may still be read from a previous call
  if (lane == 63) part[w] = inc;
  __syncthreads();
  uint32_t base = 0, all = 0;
  for (int i = 0; i < nw; ++i) {
    const uint32_t p = part[i];
    if (i < w) base += p;
    all += p;
  }
  if (total) *total = all;
  return base + inc - v;
}

// Many tiles: the histograms' exclusive prefixes over the tiles, in place, and the totals per digit.  One workgroup per 64
// digits, a wavefront per 16th of the tiles.
constexpr int PREFIX_SEGS = 16;
__global__ __launch_bounds__(64 * PREFIX_SEGS) void k_tile_prefix(uint32_t *__restrict__ hist, int nb, int nTiles, uint32_t *__restrict__ totals) {
  __shared__ uint32_t sums[PREFIX_SEGS][64];
  const int lane = threadIdx.x & 63, seg = threadIdx.x >> 6, digit = blockIdx.x * 64 + lane;
  const int per = (nTiles + PREFIX_SEGS - 1) / PREFIX_SEGS, t0 = min(nTiles, seg * per), t1 = min(nTiles, t0 + per);
  uint32_t own = 0;
  if (digit < nb)
#pragma unroll 8
    for (int t = t0; t < t1; ++t) own += hist[(size_t)t * nb + digit];
  sums[seg][lane] = own;
  __syncthreads();
  if (digit >= nb) return;
  uint32_t run = 0;
  for (int w = 0; w < seg; ++w) run += sums[w][lane];
  if (seg == PREFIX_SEGS - 1) totals[digit] = run + own;
  for (int t = t0; t < t1; t += 8) {
    uint32_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = hist[(size_t)min(t + u, t1 - 1) * nb + digit];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (t + u < t1) hist[(size_t)(t + u) * nb + digit] = run;
      run += v[u];
    }
  }
}

// Stable scatter of one digit.  The workgroup sums the tile histograms into its offset per digit (keys of smaller digits +
// keys of this digit in earlier tiles), or finds the sums ready (totals != NULL, see k_tile_prefix); inside the tile a key's
// rank is the count of its digit in earlier wavefronts (16-bit counters per wavefront, turned into prefixes) plus its rank
// inside its wavefront by ballot matching.  vin == NULL: the values are the positions themselves (first pass).
static_assert(BINS_MAX / 4 <= SORT_THREADS, "a thread serves four digits");
constexpr size_t SCATTER_LDS = (size_t)SORT_WAVES * BINS_MAX * 2 + BINS_MAX * 4 + 32 * 4;
template <int R>
__global__ __launch_bounds__(SORT_THREADS) void k_sort_scatter(const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin,
                                                               uint64_t *__restrict__ kout, uint32_t *__restrict__ vout, int N,
                                                               int shift, int dbits, int nTiles, const uint32_t *__restrict__ hist,
                                                               const uint32_t *__restrict__ totals) {
  extern __shared__ uint32_t sort_smem[];
  const int nb = 1 << dbits, half = nb / 2, quarter = nb / 4, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  uint32_t *wcnt = sort_smem;                              // [SORT_WAVES][nb/2] packed pairs of 16-bit counters
  uint32_t *offs = wcnt + SORT_WAVES * half;               // [nb]
  uint32_t *part = offs + nb;
  uint64_t key[R];
  uint32_t val[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = tile_key<R>(r);
    key[r] = i < N ? kin[i] : 0ull;
    val[r] = i < N ? (vin ? vin[i] : (uint32_t)i) : 0u;
  }
  for (int i = tid; i < SORT_WAVES * half; i += SORT_THREADS) wcnt[i] = 0u;
  // thread t < nb/4 serves digits 4t .. 4t+3
  uint32_t before[4] = {0u, 0u, 0u, 0u}, all[4] = {0u, 0u, 0u, 0u};
  if (tid < quarter && totals) {
    const uint4 b = reinterpret_cast<const uint4 *>(hist)[(size_t)blockIdx.x * quarter + tid], t = reinterpret_cast<const uint4 *>(totals)[tid];
    before[0] = b.x; before[1] = b.y; before[2] = b.z; before[3] = b.w;
    all[0] = t.x; all[1] = t.y; all[2] = t.z; all[3] = t.w;
  } else if (tid < quarter) {
    const uint4 *row = reinterpret_cast<const uint4 *>(hist) + tid;
    for (int t0 = 0; t0 < nTiles; t0 += 16) {  // 16 loads in flight, whatever the remainder
      uint4 x[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) x[u] = row[(size_t)min(t0 + u, nTiles - 1) * quarter];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int t = t0 + u;
        const uint32_t c[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          all[j] += t < nTiles ? c[j] : 0u;
          before[j] += t < (int)blockIdx.x ? c[j] : 0u;
        }
      }
    }
  }
  uint32_t ex = block_exclusive_scan(all[0] + all[1] + all[2] + all[3], part, nullptr);
  if (tid < quarter) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      offs[4 * tid + j] = ex + before[j];
      ex += all[j];
    }
  }
  __syncthreads();
  uint16_t *mine = reinterpret_cast<uint16_t *>(wcnt + w * half);
  uint32_t rank[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool valid = tile_key<R>(r) < N;
    const uint32_t digit = (uint32_t)(key[r] >> shift) & (uint32_t)(nb - 1);
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < dbits; ++b) {
      const bool bit = (digit >> b) & 1u;
      const uint64_t m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    const uint32_t below = (uint32_t)__popcll(peers & ((1ull << lane) - 1ull)), base = mine[digit];
    rank[r] = base + below;
    __builtin_amdgcn_wave_barrier();
    if (valid && below == 0) mine[digit] = (uint16_t)(base + __popcll(peers));
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  if (tid < quarter) {
    uint2 c[SORT_WAVES], run = make_uint2(0u, 0u);
#pragma unroll
    for (int ww = 0; ww < SORT_WAVES; ++ww) c[ww] = *reinterpret_cast<const uint2 *>(wcnt + ww * half + 2 * tid);
#pragma unroll
    for (int ww = 0; ww < SORT_WAVES; ++ww) {
      *reinterpret_cast<uint2 *>(wcnt + ww * half + 2 * tid) = run;
      run.x += c[ww].x;  // (no 16-bit half reaches 2^16: a tile has at most 8192 keys)
      run.y += c[ww].y;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (tile_key<R>(r) >= N) continue;
    const uint32_t digit = (uint32_t)(key[r] >> shift) & (uint32_t)(nb - 1);
    const uint32_t pos = offs[digit] + mine[digit] + rank[r];
    kout[pos] = key[r];
    vout[pos] = val[r];
  }
}

struct CsrOut {
  int32_t *perm, *inv_perm, *tok_item, *tok_cmp, *tok_slc, *tok_win;
  int32_t *cmp_start, *slc_start, *win_start, *slc_child_start, *cmp_slc, *cmp_batch, *slc_batch, *item_start;
};

// Block ids are running counts of block heads (a token whose key prefix differs from its predecessor's) at the three
// granularities.  Two launches: per-tile head counts, then every tile sums the counts before it, numbers its own tokens
// and writes all per-token and per-block arrays.
constexpr int CSR_TILE = 512;
struct Heads { bool c, s, w; };

// Where the blocks begin and which item a sorted position belongs to, for the two kinds of partition.
// Voxel grid: sorted (item << item_shift | Morton) keys; a block of side m is a change of the key above 3*log2(m) bits.
struct GridSrc {
  const uint64_t *ks;
  int sc, ss, sw, item_shift;
  __device__ Heads heads(int i) const {
    const uint64_t k = ks[i], p = i == 0 ? 0ull : ks[i - 1];
    const bool first = i == 0;
    return Heads{first || (k >> sc) != (p >> sc), first || (k >> ss) != (p >> ss), first || (k >> sw) != (p >> sw)};
  }
  __device__ int item(int i) const { return (int)(ks[i] >> item_shift); }
  __device__ int32_t source(int i, const int32_t *perm) const { return perm[i]; }  // written by the sort
};
// Sequences: the caller's order is the token order; blocks are runs of lc / ls / lw tokens counted from the start of
// each sequence (the last one of a sequence may be shorter).
struct SeqSrc {
  const int32_t *offs;
  int B, lc, ls, lw;
  __device__ int item(int i) const {
    int lo = 0, hi = B;  // offs[lo] <= i < offs[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (offs[mid] <= i) lo = mid; else hi = mid;
    }
    return lo;
  }
  __device__ Heads heads(int i) const {
    const int pos = i - offs[item(i)];
    return Heads{pos % lc == 0, pos % ls == 0, pos % lw == 0};
  }
  __device__ int32_t source(int i, int32_t *perm) const { return perm[i] = i; }
};

template <class Src>
__global__ __launch_bounds__(CSR_TILE) void k_csr_count(Src src, int N, int nTiles, uint32_t *__restrict__ tile_cnt) {
  __shared__ uint32_t cnt[3];
  if (threadIdx.x < 3) cnt[threadIdx.x] = 0;
  __syncthreads();
  const int i = blockIdx.x * CSR_TILE + threadIdx.x;
  Heads h{false, false, false};
  if (i < N) h = src.heads(i);
  const uint64_t bc = __ballot(h.c), bs = __ballot(h.s), bw = __ballot(h.w);
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(&cnt[0], (uint32_t)__popcll(bc));
    atomicAdd(&cnt[1], (uint32_t)__popcll(bs));
    atomicAdd(&cnt[2], (uint32_t)__popcll(bw));
  }
  __syncthreads();
  if (threadIdx.x < 3) tile_cnt[threadIdx.x * nTiles + blockIdx.x] = cnt[threadIdx.x];
}

// Many tiles: exclusive prefixes of the three count rows over the tiles, in place; a workgroup per row.
__global__ __launch_bounds__(1024) void k_csr_prefix(uint32_t *__restrict__ tile_cnt, int nTiles) {
  __shared__ uint32_t part[1024 / 64 + 1];
  uint32_t *row = tile_cnt + (size_t)blockIdx.x * nTiles, carry = 0;
  for (int t0 = 0; t0 < nTiles; t0 += 1024) {
    const int t = t0 + threadIdx.x;
    const uint32_t v = t < nTiles ? row[t] : 0u;
    uint32_t sum;
    const uint32_t ex = block_exclusive_scan(v, part, &sum);
    if (t < nTiles) row[t] = carry + ex;
    carry += sum;
  }
}

template <class Src>
__global__ __launch_bounds__(CSR_TILE) void k_csr_write(Src src, int N, int B, int nTiles, const int32_t *__restrict__ offs,
                                                        const uint32_t *__restrict__ tile_cnt, bool summed, CsrOut o, int32_t *meta) {
  __shared__ uint32_t part[CSR_TILE / 64 + 1];
  const int i = blockIdx.x * CSR_TILE + threadIdx.x;
  for (int j = i; j <= B; j += gridDim.x * CSR_TILE) o.item_start[j] = offs[j];
  Heads h{false, false, false};
  if (i < N) h = src.heads(i);
  // inclusive head counts up to and including token i: heads of earlier tiles + heads of this tile
  uint32_t base[3];
#pragma unroll
  for (int x = 0; x < 3; ++x) {
    if (summed) {
      base[x] = tile_cnt[x * nTiles + blockIdx.x];
      continue;
    }
    uint32_t c = 0;
    for (int t = threadIdx.x; t < (int)blockIdx.x; t += CSR_TILE) c += tile_cnt[x * nTiles + t];
    (void)block_exclusive_scan(c, part, &base[x]);
  }
  const int idc = (int)(base[0] + block_exclusive_scan(h.c, part, nullptr) + h.c) - 1;
  const int ids = (int)(base[1] + block_exclusive_scan(h.s, part, nullptr) + h.s) - 1;
  const int idw = (int)(base[2] + block_exclusive_scan(h.w, part, nullptr) + h.w) - 1;
  if (i >= N) return;
  const int item = src.item(i);
  const int pitem = i == 0 ? -1 : src.item(i - 1);
  const int32_t from = src.source(i, o.perm);
  o.inv_perm[from] = i;
  o.tok_item[i] = item;
  o.tok_cmp[i] = idc;
  o.tok_slc[i] = ids;
  o.tok_win[i] = idw;
  if (h.c) { o.cmp_start[idc] = i; o.cmp_slc[idc] = ids; }
  if (h.s) { o.slc_start[ids] = i; o.slc_child_start[ids] = idc; }
  if (h.w) o.win_start[idw] = i;
  for (int it = pitem + 1; it <= item; ++it) { o.cmp_batch[it] = idc; o.slc_batch[it] = ids; }
  if (i == N - 1) {
    const int Nc = idc + 1, Ns = ids + 1, Nw = idw + 1;
    o.cmp_start[Nc] = N; o.slc_start[Ns] = N; o.win_start[Nw] = N; o.slc_child_start[Ns] = Nc;
    for (int it = item + 1; it <= B; ++it) { o.cmp_batch[it] = Nc; o.slc_batch[it] = Ns; }
    meta[META_NC] = Nc; meta[META_NS] = Ns; meta[META_NW] = Nw;
  }
}

// Validation of the batch offsets alone (the sequence builder has no coordinates to read).
__global__ void k_check_offsets(const int32_t *__restrict__ offs, int N, int B, int32_t *meta) {
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j <= B; j += gridDim.x * blockDim.x) {
    const int o = offs[j];
    const bool bad = (j == 0 && o != 0) || (j == B && o != N) || (j > 0 && o < offs[j - 1]) || o < 0 || o > N;
    if (bad) atomicOr(&meta[META_ERR], 1);
  }
}

// Largest per-item block counts and per-block token counts, and the tokens in long selection blocks (integer max and sum: order
// independent), then the counts to the host:
// the workgroup that finishes last copies them (and the error bits of the tiles) into pinned memory.
constexpr int MAX_THREADS = 512;
__global__ __launch_bounds__(MAX_THREADS) void k_maxima(CsrOut o, int B, const int32_t *__restrict__ err, int n_err, int32_t *meta,
                                                        int32_t *host_meta) {
  __shared__ int best[7], last;
  if (threadIdx.x < 7) best[threadIdx.x] = 0;
  __syncthreads();
  const int Nc = meta[META_NC], Ns = meta[META_NS], Nw = meta[META_NW], i0 = blockIdx.x * MAX_THREADS + threadIdx.x;
  const int stride = gridDim.x * MAX_THREADS;
  int m[5] = {0, 0, 0, 0, 0}, sum[2] = {0, 0};  // in the order META_SMAX .. META_CMP_TOK, META_SLC_128, META_SLC_256
  for (int i = i0; i < B; i += stride) {
    m[0] = max(m[0], o.slc_batch[i + 1] - o.slc_batch[i]);
    m[1] = max(m[1], o.cmp_batch[i + 1] - o.cmp_batch[i]);
  }
  for (int i = i0; i < Ns; i += stride) {
    const int len = o.slc_start[i + 1] - o.slc_start[i];
    m[2] = max(m[2], len);
    sum[0] += len > 128 ? len : 0;
    sum[1] += len > 256 ? len : 0;
  }
  for (int i = i0; i < Nw; i += stride) m[3] = max(m[3], o.win_start[i + 1] - o.win_start[i]);
  for (int i = i0; i < Nc; i += stride) m[4] = max(m[4], o.cmp_start[i + 1] - o.cmp_start[i]);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {  // (seven independent chains of lane exchanges)
#pragma unroll
    for (int x = 0; x < 5; ++x) m[x] = max(m[x], __shfl_xor(m[x], off));
    sum[0] += __shfl_xor(sum[0], off);
    sum[1] += __shfl_xor(sum[1], off);
  }
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int x = 0; x < 5; ++x) atomicMax(&best[x], m[x]);
    if (sum[0]) atomicAdd(&best[5], sum[0]);
    if (sum[1]) atomicAdd(&best[6], sum[1]);
  }
  __syncthreads();
  // (device-scope atomics meet in memory; their returned values are waited for, so they are done before META_DONE counts
  // this workgroup, without a fence that would write back the caches)
  if (threadIdx.x < 5) {
    const int old = atomicMax(&meta[META_SMAX + threadIdx.x], best[threadIdx.x]);
    asm volatile("" : : "v"(old));
  } else if (threadIdx.x >> 1 == 32 && best[5 + (threadIdx.x & 1)]) {  // (two lanes of the second wavefront, beside the maxima)
    const int old = atomicAdd(&meta[META_SLC_128 + (threadIdx.x & 1)], best[5 + (threadIdx.x & 1)]);
    asm volatile("" : : "v"(old));
  }
  __syncthreads();
  if (threadIdx.x == 0) last = atomicAdd(&meta[META_DONE], 1) == (int)gridDim.x - 1;
  __syncthreads();
  if (!last) return;
  int e = 0;
  for (int i = threadIdx.x; i < n_err; i += MAX_THREADS) e |= err[i];
  if (e) {
    const int old = atomicOr(&meta[META_ERR], e);
    asm volatile("" : : "v"(old));
  }
  __syncthreads();
  if (threadIdx.x < META_N) host_meta[threadIdx.x] = atomicAdd(&meta[threadIdx.x], 0);
}

// Read-out of one index array (a launch costs less than a runtime copy of this size).
__global__ __launch_bounds__(256) void k_copy(const int32_t *__restrict__ src, size_t n, int32_t *__restrict__ dst) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) dst[i] = src[i];
}

// Pinned slots through which the kernels hand their counts to the host (one per build in progress).
class PinnedSlots {
 public:
  static PinnedSlots &get() {
    static PinnedSlots *p = new PinnedSlots();
    return *p;
  }
  int32_t *take() {
    std::lock_guard<std::mutex> l(mu_);
    if (free_.empty()) {
      void *p = nullptr;
      if (hipHostMalloc(&p, SLOT_INTS * 4 * 32, hipHostMallocPortable) != hipSuccess) return nullptr;
      for (int i = 0; i < 32; ++i) free_.push_back((int32_t *)p + i * SLOT_INTS);
    }
    int32_t *s = free_.back();
    free_.pop_back();
    return s;
  }
  void give(int32_t *s) {
    std::lock_guard<std::mutex> l(mu_);
    free_.push_back(s);
  }

 private:
  static constexpr int SLOT_INTS = 32;
  static_assert(META_INTS <= SLOT_INTS, "a slot holds the counts");
  std::mutex mu_;
  std::vector<int32_t *> free_;
};

// Kernels of the sort for R keys per thread.  k1: second key array; the sorted keys end in kdst, the caller indices in vdst.
template <int R>
void launch_sort(const int32_t *coords, const int32_t *offs, int N, int B, int G, int bits, int total_bits, uint64_t *k0, uint64_t *k1,
                 uint32_t *v1, uint64_t *kdst, uint32_t *vdst, uint32_t *hist, uint32_t *totals, int32_t *err, int32_t *meta, int nTiles,
                 hipStream_t s) {
  static std::once_flag once;
  std::call_once(once, [] {
    (void)hipFuncSetAttribute((const void *)k_sort_scatter<R>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)SCATTER_LDS);
  });
  const int passes = (total_bits + DIGIT_BITS_MAX - 1) / DIGIT_BITS_MAX;
  const int dbits = (total_bits + passes - 1) / passes;
  const size_t lds = ((size_t)SORT_WAVES * 2 + 4) * ((size_t)1 << dbits) + 32 * 4;
  k_keys_hist<R><<<nTiles, SORT_THREADS, 0, s>>>(coords, offs, N, B, G, bits, dbits, k0, hist, err, meta);
  uint64_t *kin = k0, *kalt = k1;
  uint32_t *vin = nullptr, *valt = v1, *vspare = v1 + N;
  for (int p = 0; p < passes; ++p) {
    const bool final = p == passes - 1;
    uint64_t *ko = final ? kdst : kalt;
    uint32_t *vo = final ? vdst : valt;
    if (p > 0) k_sort_hist<R><<<nTiles, SORT_THREADS, 0, s>>>(kin, N, p * dbits, dbits, hist);
    if (totals) k_tile_prefix<<<((1 << dbits) + 63) / 64, 64 * PREFIX_SEGS, 0, s>>>(hist, 1 << dbits, nTiles, totals);
    k_sort_scatter<R><<<nTiles, SORT_THREADS, lds, s>>>(kin, vin, ko, vo, N, p * dbits, dbits, nTiles, hist, totals);
    kalt = kin;
    kin = ko;
    vin = vo;
    uint32_t *t = valt; valt = vspare; vspare = t;
  }
}

}  // namespace

// Up to so many tokens every workgroup sums what the tiles before it counted; that work grows with the square of the tile count,
// so beyond it a launch forms the prefixes once (sort and block arrays with the sums, with the prefixes: 83 + 33 and 89 + 31 us at
// 500 k tokens, 102 + 53 and 98 + 46 at 1 M, 188 + 111 and 168 + 77 at 2 M, 3591 + 1883 and 1441 + 666 at 16 M).
constexpr int SUM_TOKENS_MAX = 1 << 20;

// Common part of the two builders: grid_mode = voxel partition (sort by Morton key), else sequences in caller order.
static int build_handle(const ssa_params_t *p, const int32_t *coords, const int32_t *batch_offsets, bool grid_mode,
                        hipStream_t stream, ssa_blocks_t **out) {
  const int N = p->n_tokens, B = p->n_batch;
  int bits = 1;
  while ((1 << bits) < p->grid) ++bits;
  int item_bits = 0;
  while ((1ll << item_bits) < (long long)B) ++item_bits;

  ssa_blocks *h = new ssa_blocks();
  h->N = N; h->B = B; h->G = p->grid; h->m_cmp = p->m_cmp; h->m_slc = p->m_slc; h->m_win = p->m_win;
  h->bits = grid_mode ? bits : 0;
  h->dims = grid_mode ? 3 : 1;
  if (hipGetDevice(&h->device) != hipSuccess) { delete h; return SSA_ERR_HIP; }
  DevicePool &pool = DevicePool::get();
  const size_t n1 = (size_t)N + 1;
  const size_t ints = 2 * (size_t)N + 6 * (size_t)N + 4 * n1 + (size_t)N + 3 * ((size_t)B + 1) + 64;
  h->base = pool.take(h->device, ints * sizeof(int32_t), &h->bytes);
  if (!h->base) { delete h; return SSA_ERR_HIP; }
  int32_t *w = (int32_t *)h->base;
  auto take = [&](size_t n) { int32_t *r = w; w += n; return r; };
  h->sorted_keys = (uint64_t *)take(2 * (size_t)N);  // first: the allocation's alignment serves the 8-byte keys
  h->perm = take(N); h->inv_perm = take(N); h->tok_item = take(N); h->tok_cmp = take(N); h->tok_slc = take(N);
  h->tok_win = take(N); h->cmp_start = take(n1); h->slc_start = take(n1); h->win_start = take(n1);
  h->slc_child_start = take(n1); h->cmp_slc = take(N); h->cmp_batch = take(B + 1); h->slc_batch = take(B + 1);
  h->item_start = take(B + 1);

  // keys per thread of the sort: about 32 tiles, whose histograms every scatter workgroup reads (16 and 64 tiles: +2, +3 %)
  int R = 1;
  while (R < 16 && (long long)N > 32ll * SORT_THREADS * R) R *= 2;
  const int nTiles = N > 0 ? (N + SORT_THREADS * R - 1) / (SORT_THREADS * R) : 1;
  const int csrTiles = N > 0 ? (N + CSR_TILE - 1) / CSR_TILE : 1;
  const size_t key_b = align_up((size_t)N * 8, 256), val_b = align_up((size_t)2 * N * 4, 256);
  const size_t hist_b = align_up((size_t)BINS_MAX * nTiles * 4, 256), err_b = align_up((size_t)nTiles * 4, 256);
  const size_t cnt_b = align_up((size_t)3 * csrTiles * 4, 256);
  const size_t tmp_bytes = (grid_mode ? 2 * key_b + val_b + hist_b + BINS_MAX * 4 : 0) + err_b + cnt_b + 256;
  size_t tmp_got = 0;
  void *tmp = pool.take(h->device, tmp_bytes, &tmp_got);
  int32_t *host_meta = PinnedSlots::get().take();
  // nothing goes back to the pools while the stream may still use it
  auto fail = [&](int code) {
    const bool idle = hipStreamSynchronize(stream) == hipSuccess;
    if (tmp) { if (idle) pool.give(h->device, tmp, tmp_got); else (void)hipFree(tmp); }
    if (idle) pool.give(h->device, h->base, h->bytes); else (void)hipFree(h->base);
    if (host_meta && idle) PinnedSlots::get().give(host_meta);
    delete h;
    return code;
  };
  if (!tmp || !host_meta) return fail(SSA_ERR_HIP);
  char *tp = (char *)tmp;
  auto tmp_take = [&](size_t n) { char *r = tp; tp += n; return r; };
  int32_t *err = (int32_t *)tmp_take(err_b);
  uint32_t *tile_cnt = (uint32_t *)tmp_take(cnt_b);
  int32_t *meta = (int32_t *)tmp_take(256);
  CsrOut o{h->perm, h->inv_perm, h->tok_item, h->tok_cmp, h->tok_slc, h->tok_win, h->cmp_start, h->slc_start,
           h->win_start, h->slc_child_start, h->cmp_slc, h->cmp_batch, h->slc_batch, h->item_start};
  int n_err = 0;
  auto csr = [&](auto src) {
    k_csr_count<<<csrTiles, CSR_TILE, 0, stream>>>(src, N, csrTiles, tile_cnt);
    const bool summed = N > SUM_TOKENS_MAX;
    if (summed) k_csr_prefix<<<3, 1024, 0, stream>>>(tile_cnt, csrTiles);
    k_csr_write<<<csrTiles, CSR_TILE, 0, stream>>>(src, N, B, csrTiles, batch_offsets, tile_cnt, summed, o, meta);
  };
  if (!grid_mode || N == 0) {
    // The offsets are checked first and the result is read back before any kernel searches them: SeqSrc::item assumes
    // ascending offsets that start at 0 and end at N.
    if (hipMemsetAsync(meta, 0, 256, stream) != hipSuccess) return fail(SSA_ERR_HIP);
    k_check_offsets<<<1, 256, 0, stream>>>(batch_offsets, N, B, meta);
    if (hipMemcpyAsync(host_meta, meta, META_N * sizeof(int32_t), hipMemcpyDeviceToHost, stream) != hipSuccess) return fail(SSA_ERR_HIP);
    if (hipStreamSynchronize(stream) != hipSuccess) return fail(SSA_ERR_HIP);
    if (host_meta[META_ERR] & 1) return fail(SSA_ERR_BAD_OFFSETS);
  }
  if (N == 0) {  // no tokens: every start array is a single zero
    if (hipMemsetAsync(h->base, 0, ints * sizeof(int32_t), stream) != hipSuccess) return fail(SSA_ERR_HIP);
  } else if (grid_mode) {
    uint64_t *k0 = (uint64_t *)tmp_take(key_b), *k1 = (uint64_t *)tmp_take(key_b);
    uint32_t *v1 = (uint32_t *)tmp_take(val_b), *hist = (uint32_t *)tmp_take(hist_b), *totals = (uint32_t *)tmp_take(BINS_MAX * 4);
    if (N <= SUM_TOKENS_MAX) totals = nullptr;
    auto sort = [&](auto r) {
      launch_sort<decltype(r)::value>(coords, batch_offsets, N, B, p->grid, bits, 3 * bits + item_bits, k0, k1, v1, h->sorted_keys,
                                      (uint32_t *)h->perm, hist, totals, err, meta, nTiles, stream);
    };
    switch (R) {
      case 1: sort(std::integral_constant<int, 1>()); break;
      case 2: sort(std::integral_constant<int, 2>()); break;
      case 4: sort(std::integral_constant<int, 4>()); break;
      case 8: sort(std::integral_constant<int, 8>()); break;
      default: sort(std::integral_constant<int, 16>()); break;
    }
    n_err = nTiles;
    csr(GridSrc{h->sorted_keys, 3 * ilog2_exact(p->m_cmp), 3 * ilog2_exact(p->m_slc), 3 * ilog2_exact(p->m_win), 3 * bits});
  } else {
    csr(SeqSrc{batch_offsets, B, p->m_cmp, p->m_slc, p->m_win});
    if (hipMemsetAsync(h->sorted_keys, 0, (size_t)N * sizeof(uint64_t), stream) != hipSuccess) return fail(SSA_ERR_HIP);
  }
  if (N > 0) {
    const int span = N > B ? N : B, wgs = (span + 4 * MAX_THREADS - 1) / (4 * MAX_THREADS);
    k_maxima<<<wgs < 64 ? wgs : 64, MAX_THREADS, 0, stream>>>(o, B, err, n_err, meta, host_meta);
  }
  if (hipGetLastError() != hipSuccess) return fail(SSA_ERR_HIP);
  if (hipStreamSynchronize(stream) != hipSuccess) return fail(SSA_ERR_HIP);
  if (host_meta[META_ERR] & 1) return fail(SSA_ERR_BAD_OFFSETS);
  if (host_meta[META_ERR] & 2) return fail(SSA_ERR_COORD_RANGE);
  h->Nc = host_meta[META_NC]; h->Ns = host_meta[META_NS]; h->Nw = host_meta[META_NW];
  h->s_max = host_meta[META_SMAX]; h->c_max = host_meta[META_CMAX]; h->slc_tok_max = host_meta[META_SLC_TOK];
  h->win_tok_max = host_meta[META_WIN_TOK]; h->cmp_tok_max = host_meta[META_CMP_TOK];
  h->slc_tok_128 = host_meta[META_SLC_128]; h->slc_tok_256 = host_meta[META_SLC_256];
  pool.give(h->device, tmp, tmp_got);
  PinnedSlots::get().give(host_meta);
  *out = h;
  return SSA_OK;
}

extern "C" int ssa_build_blocks(const ssa_params_t *p, const int32_t *coords, const int32_t *batch_offsets,
                                void *stream_, ssa_blocks_t **out) {
  if (!p || !out) return SSA_ERR_NULL;
  *out = nullptr;
  if (p->n_tokens < 0 || p->n_batch < 1 || p->grid < 1 || p->grid > 1024) return SSA_ERR_BAD_SHAPE;
  if (p->m_cmp < 1 || p->m_slc < 1 || p->m_win < 1 || p->m_slc <= p->m_cmp || p->m_slc % p->m_cmp != 0)
    return SSA_ERR_BAD_BLOCK_SIZES;
  auto pow2 = [](int m) { return (m & (m - 1)) == 0; };
  if (!pow2(p->m_cmp) || !pow2(p->m_slc) || !pow2(p->m_win)) return SSA_ERR_UNSUPPORTED;
  if (!batch_offsets || (p->n_tokens > 0 && !coords)) return SSA_ERR_NULL;
  return build_handle(p, coords, batch_offsets, true, (hipStream_t)stream_, out);
}

extern "C" int ssa_build_blocks_1d(const ssa_params_t *p, const int32_t *batch_offsets, void *stream_,
                                   ssa_blocks_t **out) {
  if (!p || !out) return SSA_ERR_NULL;
  *out = nullptr;
  if (p->n_tokens < 0 || p->n_batch < 1) return SSA_ERR_BAD_SHAPE;
  if (p->m_cmp < 1 || p->m_slc < 1 || p->m_win < 1 || p->m_slc <= p->m_cmp || p->m_slc % p->m_cmp != 0)
    return SSA_ERR_BAD_BLOCK_SIZES;
  if (!batch_offsets) return SSA_ERR_NULL;
  return build_handle(p, nullptr, batch_offsets, false, (hipStream_t)stream_, out);
}

extern "C" int ssa_blocks_counts(const ssa_blocks_t *b, int32_t *n_cmp, int32_t *n_slc, int32_t *n_win) {
  if (!b) return SSA_ERR_NULL;
  if (n_cmp) *n_cmp = b->Nc;
  if (n_slc) *n_slc = b->Ns;
  if (n_win) *n_win = b->Nw;
  return SSA_OK;
}

extern "C" int ssa_blocks_max_slc_per_item(const ssa_blocks_t *b, int32_t *s_max) {
  if (!b || !s_max) return SSA_ERR_NULL;
  *s_max = b->s_max;
  return SSA_OK;
}

extern "C" int ssa_blocks_export(const ssa_blocks_t *b, int which, void *dst, size_t bytes, void *stream) {
  if (!b || !dst) return SSA_ERR_NULL;
  const int32_t *src = nullptr;
  size_t n = 0;
  switch (which) {
    case SSA_ARR_PERM: src = b->perm; n = b->N; break;
    case SSA_ARR_INV_PERM: src = b->inv_perm; n = b->N; break;
    case SSA_ARR_CMP_START: src = b->cmp_start; n = (size_t)b->Nc + 1; break;
    case SSA_ARR_SLC_START: src = b->slc_start; n = (size_t)b->Ns + 1; break;
    case SSA_ARR_WIN_START: src = b->win_start; n = (size_t)b->Nw + 1; break;
    case SSA_ARR_SLC_CHILD_START: src = b->slc_child_start; n = (size_t)b->Ns + 1; break;
    case SSA_ARR_CMP_BATCH: src = b->cmp_batch; n = (size_t)b->B + 1; break;
    case SSA_ARR_SLC_BATCH: src = b->slc_batch; n = (size_t)b->B + 1; break;
    case SSA_ARR_TOK_WIN: src = b->tok_win; n = b->N; break;
    default: return SSA_ERR_BAD_SHAPE;
  }
  if (bytes < n * sizeof(int32_t)) return SSA_ERR_WORKSPACE;
  if (n == 0) return SSA_OK;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev != b->device) {  // a kernel reaches another device's memory only with peer access
    SSA_HIP_TRY(hipMemcpyAsync(dst, src, n * sizeof(int32_t), hipMemcpyDeviceToDevice, (hipStream_t)stream));
    return SSA_OK;
  }
  const size_t wgs = (n + 1023) / 1024;
  k_copy<<<(unsigned)(wgs < 1024 ? wgs : 1024), 256, 0, (hipStream_t)stream>>>(src, n, (int32_t *)dst);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}

extern "C" void ssa_blocks_destroy(ssa_blocks_t *b) {
  if (!b) return;
  if (b->base) {
    // work on any stream may still read the arrays: they are kept for the next build only once the device is idle
    int dev = -1;
    if (hipGetDevice(&dev) == hipSuccess && dev == b->device && DevicePool::wait_idle())
      DevicePool::get().give(b->device, b->base, b->bytes);
    else
      (void)hipFree(b->base);
  }
  delete b;
}
