// How the work chunks of the selection kernels are ordered (sel_index.hip) and how long those of the one-pass backward are, as rules on
// the problem's sizes alone.  Host code without HIP.
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

// Query tokens per work chunk of the one-pass selection backward, for lists of `entries` tokens in all, blocks of up to `longest` keys and `heads`
// query heads per KV head.  Long chunks write fewer partial dK and dV rows and pay less for the keys they begin with, in a block of
// more than 256 keys once per segment of 256; short ones leave fewer compute units idle at the end.  So there is a number of chunks
// wanted: of four wavefronts and a few rows, some 2000; of eight, some 500; of segments, 192 of 256 tokens and twice as many of 512; fewer where
// few heads make few rows of a token.  us of the kernel, the index, the launches beside it, the sums of the partial rows and the finish, chunks
// of 128 / 256 / 512, by entries.
//   up to 128 keys, 8 heads  64k 220 / 229 / 268, 256k 432 / 448 / 496, 544k 955 / 945 / 969, 640k 951 / 947 / 953, 1.3M 2182 / 2113 / 2129, 2.2M 4823 / 4713 /
//                            4700; 16 heads of 32 256k 437 / 464 / 490, 640k 1003 / 1017 / 1051, 2.2M 5358 / 5271 / 5331
//                   2 heads  16k 65 / 72 / 78, 160k 217 / 209 / 209, 384k 257 / 242 / 234;  1: 64k 96 / 91 / 89, 192k 240 / 224 / 214, 640k 277 / 245 / 220
//   up to 256 keys, 8 heads  96k 264 / 258 / 293, 128k 367 / 383 / 470, 256k 635 / 662 / 704, 341k in three shapes 827 / 803 / 790, 640k 1517 / 1448 / 1478
//                   4 heads  40k 163 / 152 / 185, 96k 295 / 277 / 265, 480k 1392 / 1314 / 1284;  1: 32k 99 / 89 / 95, 80k 137 / 128 / 119, 480k 746 / 636 / 572
//   longer,         8 heads  40k 248 / 302 / 443, 53k (1618 keys) 1744 / 1422 / 1837, 64k 425 / 404 / 533, 137k 488 / 447 / 549, 170k 546 / 509 / 561, 224k 806 / 748 / 722,
//                            384k 1242 / 1055 / 976;  1: 16k 196 / 175 / 190, 32k 462 / 320 / 310, 53k 1500 / 892 / 635
constexpr int DKV_CHUNK_MIN = 128;
inline int one_pass_chunk_len(int longest, long long entries, int heads) {
  auto wanted = [&](int len) {
    if (longest <= 128) return 256 * (heads < 8 ? heads : 8);
    if (longest <= 256) return heads < 8 ? 150 : 560;
    return len / 256 * 48 * (heads < 4 ? heads : 4);
  };
  int len = 512;
  while (len > DKV_CHUNK_MIN && entries / len < wanted(len)) len /= 2;
  return len;
}
