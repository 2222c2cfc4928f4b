// How a weight gradient's sum over positions is cut into chunks, one block each
// per tile of the result, whose partial sums are added afterwards.  Host
// arithmetic only.  The number of chunks of N positions is not monotone in N
// (a chunk is a whole number of stages, rounded up: 128 stages give 128 chunks
// of one, 150 give 75 of two), so a workspace for up to max_batch windows is
// sized by the bounds, which grow with N and are never below the chunks of any
// smaller batch.
#pragma once

#include <algorithm>

namespace wsn {

constexpr int kTile = 64;     // output rows and columns per block of the generic forms
constexpr int kTk = 16;       // reduction depth staged per LDS step
constexpr int kDirP = 64;     // positions per stage of the matrix-core forms
constexpr int kWgradTarget = 512;   // blocks aimed at per weight-gradient launch
constexpr int kDirectTarget = 512;  // the same for the matrix-core form (two blocks per CU)

struct Chunks {
  int chunk;   // positions per chunk
  int count;   // chunks
};

// k_wgrad: M rows, Kr columns and the bias one, N positions.
inline int wgrad_bound(int M, int Kr, int N) {
  const int tiles = ((Kr + 1 + kTile - 1) / kTile) * ((M + kTile - 1) / kTile);
  return std::max(1, std::min((kWgradTarget + tiles - 1) / tiles, (N + kTile - 1) / kTile));
}
inline Chunks wgrad_chunks(int M, int Kr, int N) {
  const int most = wgrad_bound(M, Kr, N);
  const int c = ((N + most - 1) / most + kTk - 1) / kTk * kTk;
  return {c, (N + c - 1) / c};
}

// k_wgrad_direct: M rows, Cin channels with all their taps.
inline int direct_bound(int M, int Cin, int N) {
  const int tiles = ((Cin + 31) / 32) * ((M + 127) / 128);
  return std::min((N + kDirP - 1) / kDirP, std::max(1, kDirectTarget / tiles));
}
inline Chunks direct_chunks(int M, int Cin, int N) {
  const int stages = (N + kDirP - 1) / kDirP, most = direct_bound(M, Cin, N);
  const int c = (stages + most - 1) / most * kDirP;
  return {c, (N + c - 1) / c};
}

}  // namespace wsn
