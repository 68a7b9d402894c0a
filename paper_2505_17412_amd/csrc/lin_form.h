// Which tiles the projections' products run in (linear.hip), as rules on their sizes alone.  Host code without HIP.
#pragma once

constexpr int WIDE = 256;  // features and tokens of a wide tile

// Whether Y = X W^T over M tokens, F features and a contraction of K runs in tiles of 256 x 256: where the useful part of the rounds of such
// tiles, one per compute unit, is large enough.  Rounds are those of an XCD with its 32 compute units: it has every eighth stretch of 256
// tokens, with all features (12.8k tokens x 1280 features are 250 tiles, but 35 of them belong to one XCD: two rounds).  A short
// contraction has less to win: two to twelve chunks of 64, of which the first waits for memory and the last for the stores, in a single
// round for all tiles at once; the shortest one wins where the outputs, beyond the caches, are all there is.
// Tiles of 128 / of 256, us, by K and useful part.
//   1024  12.8k -> 1280 (0.49) 46.3 / 54.7, 10.7k -> 1408 (0.45) 40.4 / 55.1, 12k -> 1024 (0.73) 36.0 / 37.9, 12.8k -> 1024 (0.78) 42.6 / 37.7,
//         20k -> 1408 (0.84) and 32k -> 1280 (0.83) faster by 13 and 15 %
//    512  24k -> 1024 (0.75) 36.3 / 37.4, 20k -> 1408 (0.84) 38.4 / 39.8, 46k -> 1280 (0.88) faster by 12 %; in one round 10.7k -> 1280 (0.81)
//         23.0 / 20.0, 33k -> 384 (0.75) 20.1 / 20.5
//    256  24k -> 1024 (0.75) 22.8 / 24.4, 100k -> 1408 (0.84) 130 / 131, 46k -> 1024 (0.93) 40.9 / 38.6; in one round 12.8k -> 1024 (0.78) 16.0 / 14.3
//    128  24k -> 1024 (0.75) 17.3 / 20.0, 25k -> 2048 (1.0) 28.7 / 30.2, 62k -> 2048 (0.95, eight rounds) 71.0 / 74.0, 100k -> 1408 (0.84, ten)
//         110 / 96, 150k -> 1280 (0.95, twelve) 148 / 126
// A data gradient (gradient) is followed by the weight gradient, which takes longer behind wide tiles of it: 150k tokens, 1024 inputs, 128 outputs: the
// data gradient 98 / 94, the weight gradient behind it 131 / 145.  With a short contraction that is more than they win.  Both directions of ssa_linear_backward:
//    256 (outputs)  one round 62 / 60 (16k, 1024 inputs), two 83 / 80 (16k, 2048) and 88 / 88 (33k, 1024); four 145 / 149 (65k, 1024), ten 309 / 331 (160k), 21
//                   587 / 603 (330k); 1280 four 134 / 139, 13 369 / 375, twenty 588 / 578
//    128            ten 248 / 270 (160k, 1024), 16 421 / 440 (260k), 375 / 379 (131k, 2048), 390 / 384 (200k, 1280); 20 506 / 484 (260k), 25 553 / 529 (200k, 2048)
inline bool lin_wide(int M, int F, int K, bool gradient = false) {
  const long long tiles_m = (M + WIDE - 1) / WIDE, tiles_f = (F + WIDE - 1) / WIDE, rounds = ((tiles_m + 7) / 8 * tiles_f + 31) / 32;
  const int percent = K >= 768 ? 75 : rounds == 1 && K >= 256 ? 76 : K >= 384 ? 85 : K >= 256 ? 90 : rounds >= 9 ? 80 : 101;
  if (gradient && (K >= 256 ? K < 384 && rounds > 2 : rounds < 19)) return false;
  return 100ll * M * F >= percent * rounds * 256 * WIDE * WIDE;
}

// Splits of the token range in which the weight gradient dY^T X (d_in inputs, F outputs) runs in tiles of 256 x 256, one round of them, or 0: in
// tiles of 128, `narrow` workgroups of them, three to a compute unit.  From how many tokens a split on wide tiles win depends on what they
// are against (speed of tiles of 256 over that of 128, by tokens a split, four runs of either in turn):
//   384   rounds of tiles of 128 that end with most units idle: 1024 -> 1280 384 1.08, 800 1.21; 1408 -> 1280 384 1.20; 4096 -> 1280 384 1.02
//   384   full rounds, an odd number of tiles of 128 along the inputs, so that every XCD reads all of X: 640 -> 1024 384 1.28, 768 1.42;
//         1408 -> 256 300 0.97, 384 1.06, 768 1.43; with a useful part of 0.75 in 32 splits 384 -> 1024 384 1.09, 640 1.19, but 384 -> 2048 450 0.94
//   512   full rounds, few outputs and inputs, and with them small partial sums: 1024 -> 256 300 0.92, 450 1.02, 520 1.05; 256 -> 1280 450 1.00, 640 1.04
//   704   other full rounds: 1024 -> 1024 384 0.97, 640 1.01, 768 1.05, 1500 1.17; 2048 -> 256 384 0.92, 640 0.95, 768 0.98, 1024 1.00; 2048 -> 2048 384 0.90, 640
//         0.97, 768 1.00, 1024 1.06; 1024 -> 2048 384 0.97, 640 1.06; with a useful part of 0.75 384 -> 2048 640 1.00, 384 -> 4096 768 0.98, 1024 1.01
// A tile's idle half costs more among the outputs: useful part 0.75, full rounds, 1024 -> 384 640 0.92, 1500 0.96.
constexpr int LIN_TN_ROUND = 768;
inline int lin_tn_splits(int M, int d_in, int F, long long narrow) {
  const int tiles = (F + WIDE - 1) / WIDE * ((d_in + WIDE - 1) / WIDE), s = tiles < 4 ? 64 : 256 / tiles;
  const long long useful = (long long)F * d_in * s, whole = 256ll * WIDE * WIDE;  // of the round
  if (s < 1 || 4 * useful < 3 * whole) return 0;
  const long long narrow_rounds = (narrow + LIN_TN_ROUND - 1) / LIN_TN_ROUND;
  const bool full = 10 * useful * narrow_rounds * LIN_TN_ROUND < 12 * whole * narrow, mostly = 10 * useful >= 8 * whole;
  if (full && !mostly && F % WIDE) return 0;
  const bool scattered = d_in / 128 % 2 && (mostly || s >= 32);
  const long long line = !full || scattered ? 384 : s > 50 ? 512 : 704;
  return M >= line * s ? s : 0;
}
