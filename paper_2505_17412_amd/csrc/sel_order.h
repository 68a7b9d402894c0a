// How the work chunks of the selection kernels are ordered (sel_index.hip), as a rule on the problem's sizes alone.  Host code without
// HIP.
#pragma once

constexpr int ORDER_BINS = 8192;         // bucket counters that fit the LDS table of m_chunk_order
constexpr int ORDER_CLASSES = 8;         // classes of block lengths
constexpr int BY_LENGTH_TOKENS = 24576;

// by_length: chunks run by falling length of their block alone.  Otherwise in the order of (class of block lengths, KV head, stretch
// of `bucket` query positions): classes * heads * per_head buckets, at most ORDER_BINS.
struct SelOrder {
  bool by_length;
  int bucket, per_head, classes;
};

// In small problems by falling length, whose places the last pass of the index can write, so that the chunks that end last are short;
// in large ones by classes of length and stretches of tokens, which saves fetches of the query rows.  Times of m_slc_fwd_bc / m_slc_bwd,
// us, in the order of token stretches alone and by falling length: 2k tokens 29 / - and 26 / -; 11k 139 / - and 118 / -; 21k 145 / 491
// and 130 / 415; beyond, the classes take the place of either (figures at m_chunk_order).  Near the line the two orders are equal.  All
// kernels of forward and backward, ms, by falling length / by classes, 2 KV heads of 8 query heads: 18k tokens 2.07 / 2.06, 24k 2.81 /
// 2.83, 30k 3.77 / 3.81, 40k 5.58 / 5.80, 62k 10.24 / 10.23; ungrouped, 16 KV heads: 24k 5.02 / 5.01, 40k 8.90 / 8.86, 62k 15.5 / 15.3
// (15.9 by stretches alone, which are of 128 positions then, with eight classes of 1024); sequences 16k 1.48 / 1.44, 40k 4.10 / 4.05.
// Stretches widen until the buckets fit; from 1025 KV heads on, with one stretch a head, there are fewer classes, and beyond 8192
// heads falling length alone is left.
inline SelOrder sel_order(int n_tokens, int kv_heads) {
  SelOrder o{n_tokens <= BY_LENGTH_TOKENS || kv_heads > ORDER_BINS, 64, 0, ORDER_CLASSES};
  o.per_head = (n_tokens + o.bucket - 1) / o.bucket;
  if (o.by_length) return o;
  while ((long long)o.classes * kv_heads * o.per_head > ORDER_BINS) {
    if (o.per_head > 1) {
      o.bucket *= 2;
      o.per_head = (int)(((long long)n_tokens + o.bucket - 1) / o.bucket);
    } else {
      o.classes /= 2;
    }
  }
  return o;
}
