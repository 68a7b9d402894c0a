// How the gate predictor's forward pass runs (gate.hip), as rules on its sizes alone.  Host code without HIP.
#pragma once

// Whether, with a transposed copy of the weights, the four wavefronts of a workgroup split the contraction: where a wavefront per 32 tokens
// leaves the chip half empty, at 49152 tokens and below.  Beyond, such wavefronts run in rounds of one per SIMD (32768 tokens), and a
// split, whose time grows with the tokens alone, wins where the last round is not nearly full.  With up to 32 gate columns a split is
// never behind but for a d_model of 128, a single trip, in up to 16.  Whole / split, us, 1024 features, 36 columns: 20k tokens 27.1 / 19.4,
// 49k 42.4 / 34.3, 62k (95 % of two rounds) 43.2 / 47.1, 80k (81 % of three) 60.3 / 52.7, 115k (88 % of four) 78.0 / 73.8, 150k (92 %) 100 / 110, 250k (95 %) 154 /
// 181; 60 columns: 49k 51.1 / 46.4, 62k 51.9 / 52.6, 80k 71.9 / 69.5, 150k 128 / 131; 12 columns: 62k 28.1 / 26.6, 150k 69.6 / 69.0; 128 features, 12 columns:
// 62k 7.4 / 7.4, 150k 12.4 / 13.6.
inline bool gate_split(int N, int d_model, int column_blocks) {
  const long long round = 32768, full = (N + round - 1) / round * round;
  if (column_blocks == 1 && d_model == 128) return false;
  return column_blocks <= 2 || N <= 49152 || 100ll * N < 89 * full;
}

// Weights whose rows are whole 16-byte pieces (of the gate counts that are multiples of 3 up to 64: 24 and 48) can be read as they are.
inline bool gate_whole_pieces(int J) { return J % 8 == 0; }

// Whether they are, without a transposed copy, by wavefronts that split the contraction's trips of 128 features.  With a copy and as the rule above / as
// they are, us, 1024 features, 48 columns: 5.5k tokens 11.3 / 7.1, 20k 19.1 / 14.8, 46k 33.6 / 24.2; 24 columns 10.0 / 7.4, 15.5 / 10.0, 26.2 / 18.7; 62k
// 43.5 / 31.4, 150k 100 / 94, 250k 155 / 156.  Their time grows with the tokens alone too, and where four does not divide the trips, wavefronts idle:
//   one trip     48 columns 46k 9.6 / 9.6, 57k 11.4 / 12.4, 98k 15.5 / 20.1, 250k 30.1 / 51.7; 24 columns 115k equal, 131k 15.2 / 17.3, 250k 25.0 / 30.1
//   two          48 columns 80k 24 / 24, 98k 22.0 / 24.0, 250k 46.5 / 58.3; 24 columns 250k 37.2 / 37.2, 400k 53.6 / 56.1
//   three        48 columns (here and below) 150k 42.0 / 42.5, 250k 62.7 / 67.0, 400k 102 / 127; 24 columns 400k 85.7 / 83.5
//   four         250k 86.3 / 85.3, 400k 131 / 143;  five 197k 83.7 / 80.5, 250k 104 / 129;  six 197k 104 / 105, 250k 122 / 138;  seven 197k 120 / 113, 250k 138 / 147
//   nine         115k as they are, 131k 88.8 / 99.1, 150k 113 / 121, 250k 175 / 193;  twelve, sixteen: as they are to 250k (230 / 238, 288 / 311)
// The rounds of whole contractions that are nearly full are what wins; between them as they are is the faster from three trips on.
inline bool gate_as_is(int N, int d_model, int J) {
  const int trips = d_model / 128;
  if (!gate_whole_pieces(J)) return false;
  if (J <= 32) return trips > 2 || N <= (trips == 1 ? 114688 : 262144);
  if (trips <= 2) return N <= (trips == 1 ? 49152 : 81920);
  if (gate_split(N, d_model, (J + 15) / 16)) return true;
  if (trips % 4 == 0) return trips > 4 || N <= 262144;
  return N <= (trips > 8 && trips % 4 == 1 ? 114688 : 196608);
}
