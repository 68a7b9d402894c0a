// Device code of the two passes of the selection index that touch every entry (sel_index.hip), for workgroups of any size: kernels of
// their own, or workgroups beside those of another kernel.
#pragma once

#include "mfma_launch.h"
#include "sel_order.h"

constexpr int TILE_WORDS = POS_TILE / 32;
constexpr int ORDER_STEP = 64;             // keys per class of block lengths

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

// What the two passes take.  key_tile: selection blocks of one KV head a workgroup covers, 32 bytes of LDS each.
struct SelJob {
  SelArgs a;
  int tiles, stride, key_tile, n_bins, bins_stride;
  uint32_t *cnt, *bins, *ticket;
  ScanArgs sc;
  OrderArgs bc, dkv;
  int32_t *base, *bc_base, *list;
  uint8_t *rank;
  SelOrder ord;
  bool caller_indices;
  __host__ __device__ int parts() const { return (a.Ns + key_tile - 1) / key_tile; }
  __host__ __device__ long long workgroups() const { return (long long)tiles * a.Hkv * parts(); }
  __host__ __device__ size_t lds_bytes() const { return (size_t)(a.Ns < key_tile ? a.Ns : key_tile) * TILE_WORDS * 4; }
};
struct SelPlace { int tile, g, b0; };  // of a workgroup: tile of positions, KV head, first block

// Pass 1: entries per (key, tile).  cnt[key][stride].  Workgroup column (., 0, 0) also clears the counters of the last pass.  With
// a ticket (a word that is 0 when the kernel starts) the last workgroup goes on with passes 2 and 3, a thread per key.
template <int NT>
__device__ __forceinline__ void sel_count(const SelJob &j, const SelPlace &at, uint32_t *sel_bits) {  // sel_bits: [nb][TILE_WORDS]
  const SelArgs &a = j.a;
  const ScanArgs &sc = j.sc;
  const int tile = at.tile, g = at.g, b0 = at.b0, nb = min(j.key_tile, a.Ns - b0), n_tiles = j.tiles, stride = j.stride;
  uint32_t *cnt = j.cnt, *ticket = j.ticket;
  if (g == 0 && b0 == 0)
    for (int i = tile * NT + threadIdx.x; i < j.n_bins; i += n_tiles * NT) j.bins[i] = j.bins[j.bins_stride + i] = 0u;
  for (int i = threadIdx.x; i < nb * TILE_WORDS; i += NT) sel_bits[i] = 0u;
  __syncthreads();
  const int p0 = tile * POS_TILE, npos = min(POS_TILE, a.N - p0), ne = npos * a.T;
  for (int e0 = 0; e0 < ne; e0 += 8 * NT) {
    int b[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) b[u] = sel_block(a, p0, npos, g, e0 + u * NT + threadIdx.x);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int pl = (e0 + u * NT + (int)threadIdx.x) / a.T;
      if ((unsigned)(b[u] - b0) < (unsigned)nb) atomicOr(&sel_bits[(b[u] - b0) * TILE_WORDS + (pl >> 5)], 1u << (pl & 31));
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nb; i += NT) {
    const uint4 x = *reinterpret_cast<const uint4 *>(sel_bits + i * TILE_WORDS), y = *reinterpret_cast<const uint4 *>(sel_bits + i * TILE_WORDS + 4);
    const uint32_t count = __popc(x.x) + __popc(x.y) + __popc(x.z) + __popc(x.w) + __popc(y.x) + __popc(y.y) + __popc(y.z) + __popc(y.w);
    uint32_t *to = &cnt[((size_t)g * a.Ns + b0 + i) * stride + tile];
    if (ticket) store_shared(to, count);
    else *to = count;  // (to the next kernel; written through 60k tokens' counts take 40 us for 27)
  }
  if (!ticket || !last_workgroup(ticket, (uint32_t)j.workgroups())) return;
  for (int key = threadIdx.x; key < sc.n; key += NT) {
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
        for (int i = 0; i < 4; ++i) {
          const uint32_t own = 4 * (t0 + u) + i < n_tiles ? c[i] : 0u;
          c[i] = run;
          run += own;
        }
        if (t0 + u < n4) row[t0 + u] = make_uint4(c[0], c[1], c[2], c[3]);
      }
    }
    sc.counts[key] = run;
  }
  __syncthreads();
  scan_counts<NT>(sc);
  if (j.base) order_by_length<NT>(sc, j.base, j.bc_base);
}

// Pass 4: every entry to its place: list[start of the key + entries of earlier tiles + entries of the key before it in
// this tile].  R: rounds of 8 entries per thread (POS_TILE * T entries per tile).  keys(): where the lists lie, asked for when the entries
// are requested.
struct SelKeys {
  const int32_t *start;           // [keys + 1]
  const uint32_t *before;         // [keys][stride] entries of earlier tiles
  int stride;
  const int32_t *bc_base, *base;  // as in OrderArgs
};
template <int NT, int R, class Keys>
__device__ __forceinline__ void sel_fill(const SelJob &j, const SelPlace &place, uint32_t *sel_bits, Keys keys) {
  const SelArgs &a = j.a;
  const SelOrder &ord = j.ord;
  const int tile = place.tile, g = place.g, b0 = place.b0, nb = min(j.key_tile, a.Ns - b0);
  const int32_t *slc_start = j.sc.slc_start;
  for (int i = threadIdx.x; i < nb * TILE_WORDS; i += NT) sel_bits[i] = 0u;
  __syncthreads();
  const int p0 = tile * POS_TILE, npos = min(POS_TILE, a.N - p0);
  // set the bits of all entries of this thread (they stay in registers); an entry whose bit another one owns is dropped
  int b[8 * R];
#pragma unroll
  for (int u = 0; u < 8 * R; ++u) b[u] = sel_block(a, p0, npos, g, u * NT + threadIdx.x);
  const SelKeys k = keys();
#pragma unroll
  for (int u = 0; u < 8 * R; ++u) {
    const int pl = (u * NT + (int)threadIdx.x) / a.T;
    const uint32_t bit = 1u << (pl & 31);
    if ((unsigned)(b[u] - b0) >= (unsigned)nb) b[u] = -1;
    else if (atomicOr(&sel_bits[(b[u] - b0) * TILE_WORDS + (pl >> 5)], bit) & bit) b[u] = -1;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 8 * R; ++u) {
    if (b[u] < 0) continue;
    const int e = u * NT + (int)threadIdx.x, pl = e / a.T;
    const uint32_t *w = sel_bits + (b[u] - b0) * TILE_WORDS;
    uint32_t before = __popc(w[pl >> 5] & ((1u << (pl & 31)) - 1u));
#pragma unroll
    for (int x = 0; x < TILE_WORDS - 1; ++x) before += x < (pl >> 5) ? __popc(w[x]) : 0u;
    const int key = g * a.Ns + b[u];
    const int r = (int)(k.before[(size_t)key * k.stride] + before), at = k.start[key] + r;
    j.list[at] = j.caller_indices ? a.perm[p0 + pl] : p0 + pl;
    j.rank[at] = (uint8_t)(e - pl * a.T);
    auto first = [&](const OrderArgs &o, const int32_t *base) {
      if (!o.order || r % o.chunk_len != 0) return;
      const int c = r / o.chunk_len;
      if (base) o.order[base[key] + c] = ChunkRef{key, c, at, min(o.chunk_len, k.start[key + 1] - at)};
      else {
        const int cls = ord.classes - 1 - min((slc_start[b[u] + 1] - slc_start[b[u]]) / ORDER_STEP, ord.classes - 1);
        const int bin = (cls * a.Hkv + g) * ord.per_head + (p0 + pl) / ord.bucket;
        o.slot[o.chunk_start[key] + c] = make_int4(bin, (int)atomicAdd(&o.bins[bin], 1u), key, c);
      }
    };
    first(j.bc, k.bc_base);
    first(j.dkv, k.base);
  }
}
// After the three passes before it.
__device__ inline SelKeys sel_scanned(const SelJob &j, const SelPlace &at) { return SelKeys{j.sc.start, j.cnt + at.tile, j.stride, j.bc.base, j.dkv.base}; }

// Host side (sel_index.hip): what the passes take, and the passes one by one; `beside`: for sel_beside.
SelJob sel_index_job(const int32_t *idx, const int32_t *perm, const int32_t *slc_start, int N, int Hkv, int T, int Ns, const SelIndex &x,
                     bool caller_indices, bool want_bc_order, bool want_dkv_order, bool beside);
int sel_index_count(const SelJob &j, hipStream_t s);
int sel_index_scan(const SelJob &j, hipStream_t s);
int sel_index_fill(const SelJob &j, hipStream_t s);
int sel_index_order(const SelJob &j, hipStream_t s);

// A pass as the first workgroups of another kernel's launch, with 512 blocks and 16 KB of LDS each.  The passes wait for memory on few
// compute units, so that up to 3 workgroups per 2 compute units cost what they stand beside next to nothing.  Forward and backward with
// the backward's index apart / beside its pre-pass and dQ kernel, us: 5k tokens 392 / 374, 11k 944 / 924, 21k in three shapes (168 workgroups)
// 1287 / 1275, a layer of 46k (360) 7088 / 7080.  Beyond, they take from the others what they save: pre-pass, dQ kernel and index of 62k (488)
// 1293 / 1293, of sequences of 65k in 64-token blocks (1024) 1020 / 1018, of 147k 2573 / 2700.  Entries of a row beyond 16 take more
// registers than the dQ kernel has.  (Beside the forward's window branch, whose workgroups have 128 threads: 2k tokens 83 / 91, 11k 273 / 274.)
constexpr int SEL_BESIDE_KEYS = 512, SEL_BESIDE_T = 16, SEL_BESIDE_MOST = 384;
constexpr size_t SEL_COUNT_LDS = 1024;  // what sel_count takes besides its bits, at most
enum class SelPass { none, count, fill };
struct SelBeside {
  SelJob j;
  SelPass pass;
  int n;  // workgroups
};
inline SelBeside sel_alone() { return SelBeside{SelJob{}, SelPass::none, 0}; }
inline SelBeside sel_pass(const SelJob &j, SelPass pass) { return SelBeside{j, pass, (int)j.workgroups()}; }
inline bool sel_beside_fits(int N, int Hkv, int T, int Ns) {
  return T <= SEL_BESIDE_T && ((long long)N + POS_TILE - 1) / POS_TILE * Hkv * ((Ns + SEL_BESIDE_KEYS - 1) / SEL_BESIDE_KEYS) <= SEL_BESIDE_MOST;
}
template <int NT, bool COUNT, bool FILL>  // the passes that a kernel may have beside it
__device__ __forceinline__ void sel_beside(const SelBeside &b, int wg, void *lds) {
  const SelJob &j = b.j;
  const SelPlace at{wg % j.tiles, wg / j.tiles % j.a.Hkv, wg / j.tiles / j.a.Hkv * j.key_tile};
  if constexpr (COUNT)
    if (b.pass == SelPass::count) return sel_count<NT>(j, at, (uint32_t *)lds);
  if constexpr (FILL) {
    sel_fill<NT, POS_TILE * SEL_BESIDE_T / 8 / NT>(j, at, (uint32_t *)lds, [&] { return sel_scanned(j, at); });
  }
}
