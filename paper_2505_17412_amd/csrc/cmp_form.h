// How the compression branch of the matrix-core forward is run (mfma_fwd.hip), as a rule on head dimension, heads per KV head and the
// largest number of selection blocks of an item, with the LDS of its kernels.  Host code without HIP.
#pragma once

#include <stddef.h>

// Blocks of an item whose scores a wavefront holds in registers for the top-k search; more are searched in T rounds over LDS.  With
// 1024 here: one sequence of 72k tokens (1125 blocks) 5090 us for 3320, 131k (2048) 26900 for 11600 (m_cmp_fwd of that time).
constexpr int TOPK_IN_REGISTERS = 4096;
constexpr int CMP_ONE_BLOCKS = 1024;  // the longest score rows m_cmp_fwd takes
constexpr size_t tile_bytes(int D) { return (size_t)64 * D; }  // 32 rows of D bf16

// LDS plan of m_cmp_fwd (bytes): two stages of two tiles | repeat flag, padding | lse per query row | per token its first pooled key,
// the one behind its last and the first score of its item | scores [tokens][s_max]
inline size_t cmp_lds_bytes(int D, int nw, int hs, int s_max) {
  const int tw = 32 * nw / hs;
  return 4 * tile_bytes(D) + 16 + ((size_t)32 * nw + 3 * tw + (size_t)tw * s_max) * 4;
}
// LDS plan of m_cmp_scores (bytes): two stages of st tiles | tokens as above | scores of cw groups of 32 rows | top-k marks [nw][words]
inline size_t scores_lds_bytes(int D, int hs, int cw, int nw, int st, int s_max) {
  const int tw = 32 / hs * cw;
  const size_t marks = s_max > TOPK_IN_REGISTERS ? (size_t)nw * ((s_max + 31) / 32) * 4 : 0;
  return 2 * st * tile_bytes(D) + (3 * tw + (size_t)tw * s_max) * 4 + marks;
}

constexpr size_t LDS_CU = 160 * 1024, LDS_GRANULE = 1280;  // of a compute unit; what a workgroup's share is rounded up to
// How the compression branch is run.
//  one_kernel (m_cmp_fwd): 4 heads per KV head or more, where its score rows leave a compute unit the wavefronts its registers allow, 12
//    (8 at head_dim 128).  A second launch, and the query rows read again, cost small problems 2 to 8 us (8 heads of 64, 11k tokens, 146
//    blocks: 109 us, 117 in two kernels; 4 heads 130, 137); larger ones are equal (8 heads, 25k, 176 blocks: 267, 270); beyond the line
//    wavefronts are missing (25k, 573 blocks: 718, 602; 60k, heads of 128, 938 blocks: 3220, 2260).  A wavefront searches the top-k of the
//    tokens in its 32 rows one after the other, which tells where there is little else: ungrouped heads, 700 tokens 52 us, 27 in two
//    kernels; 2 heads, 20k 401, 333; 4 heads, 3k tokens, 47 blocks 25.6, 24.5.
//  tiles_in_lds (m_cmp_scores): two groups of 32 query rows by two wavefronts each, as long as their score rows leave as many wavefronts.
//  own_tiles_4, own_tiles_8 (m_cmp_scores, every wavefront loads its own tiles): beyond that, and always for ungrouped heads, one group by
//    four wavefronts, or by eight where fewer than three workgroups of four fit.  d = 64, tiles in LDS / own by four: 4 heads, 573 blocks
//    (12 wavefronts) 776 / 816 us, 614 (8) 1570 / 1389; 8 heads, 1125 blocks (12) 2090 / 2260, 1563 (8) 4560 / 4420; ungrouped, 143 blocks
//    150 / 136.  d = 128, 8 heads, 1125 blocks (8) 3590 / 4450, 1563 (4) 9060 / 8100.  By four / eight: 4 heads, 1563 blocks (three
//    workgroups of four) 5280 / 5200, 2048 (two) 10120 / 8560.
// One kernel with 16 query columns per wavefront, the form before 32 columns: 25k tokens, 573 blocks 683 us (608 now), one sequence of 60k
// 1420 (1297), 131k 27000 (7370), 160k 40400 (10800); heads of 128, 60k 2480 (2257), 131k 31300 (13300); 4 heads, 60k 2120 (1670); ungrouped 20k
// 718 (488).  Under some 3k tokens it was faster by up to 4 us (2k tokens 17.2, now 18.3: there is one wavefront per SIMD, and it has
// twice the columns), which fewer launches around it make up for.
constexpr int cmp_wavefronts(int D) { return D <= 64 ? 12 : 8; }
inline int cmp_workgroups(size_t lds) { return (int)(LDS_CU / ((lds + LDS_GRANULE - 1) / LDS_GRANULE * LDS_GRANULE)); }
enum class CmpForm { one_kernel, tiles_in_lds, own_tiles_4, own_tiles_8 };
inline CmpForm cmp_form(int D, int hs, int s_max) {
  auto full = [&](size_t lds) { return cmp_workgroups(lds) * 4 >= cmp_wavefronts(D); };  // (workgroups of four wavefronts)
  if ((hs >= 8 || (hs == 4 && s_max > 64)) && s_max <= CMP_ONE_BLOCKS && full(cmp_lds_bytes(D, 4, hs, s_max))) return CmpForm::one_kernel;
  if (hs >= 2 && full(scores_lds_bytes(D, hs, 2, 4, 2, s_max))) return CmpForm::tiles_in_lds;
  return cmp_workgroups(scores_lds_bytes(D, hs, 1, 4, 0, s_max)) >= 3 ? CmpForm::own_tiles_4 : CmpForm::own_tiles_8;
}
// Whether m_cmp_fwd can count the selections of every one of n_blocks blocks beside its score rows, for nothing.
inline bool cmp_counts(int D, int hs, int s_max, int n_blocks) {
  return cmp_form(D, hs, s_max) == CmpForm::one_kernel && cmp_workgroups(cmp_lds_bytes(D, 4, hs, s_max) + (size_t)n_blocks * 4) * 4 >= cmp_wavefronts(D);
}

// Whether the score rows of an item's selection blocks fit the matrix-core forward: 64 query rows of them beside two stages of two key
// tiles, top-k marks and 1 KB, in 150 KB.  (The kernels above need half of the rows at most; the line stands where the path has always
// ended, as calls beyond it that only this path serves are refused.)
inline bool cmp_rows_fit(int D, int hs, int s_max) {
  const size_t words = (size_t)(64 / hs) * s_max + 4 * ((s_max + 31) / 32) + 256;
  return 4 * tile_bytes(D) + 32 + words * 4 <= 150 * 1024;
}
