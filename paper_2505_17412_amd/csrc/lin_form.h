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
inline bool lin_wide(int M, int F, int K) {
  const long long tiles_m = (M + WIDE - 1) / WIDE, tiles_f = (F + WIDE - 1) / WIDE, rounds = ((tiles_m + 7) / 8 * tiles_f + 31) / 32;
  const int percent = K >= 768 ? 75 : rounds == 1 && K >= 256 ? 76 : K >= 384 ? 85 : K >= 256 ? 90 : rounds >= 9 ? 80 : 101;
  return 100ll * M * F >= percent * rounds * 256 * WIDE * WIDE;
}
