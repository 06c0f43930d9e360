// Pieces of rows with the same column runs (find_runs), shared by the transpose
// and the lockstep products: consecutive rows inside a 64-row group that hold the
// same runs are one dense block per run.
#pragma once

#include "common.h"

namespace rfmls {

constexpr int kPieceRows = 64;

// Group g's pieces, by one wavefront (lane = row of the group): bit r of *starts is
// set where row r starts a piece (the group's first row, and every row whose runs
// differ from the row before), *lives has the rows that exist, and *wrong is
// nonzero when a row has no run description or a run leaves the columns.
__device__ __forceinline__ void group_pieces(int64_t g, int64_t rows, int64_t ncols, const int32_t* __restrict__ nrun,
                                             const int32_t* __restrict__ rcol, const int32_t* __restrict__ rend,
                                             unsigned long long* starts, unsigned long long* lives,
                                             unsigned long long* wrong) {
  const int lane = threadIdx.x & 63;
  const int64_t row = g * kPieceRows + lane;
  const bool live = row < rows;
  const int k = live ? nrun[row] : 0;
  bool start = live && lane == 0;
  bool bad = k < 0;
  if (live && k >= 0) {
    int32_t off = 0;
    const bool cmp = lane > 0;
    if (cmp && nrun[row - 1] != k) start = true;
    for (int q = 0; q < k; ++q) {
      const int32_t c = rcol[row * kMaxRuns + q], e = rend[row * kMaxRuns + q];
      bad |= c < 0 || (int64_t)c + (e - off) > ncols;
      off = e;
      if (cmp && !start && (rcol[(row - 1) * kMaxRuns + q] != c || rend[(row - 1) * kMaxRuns + q] != e)) start = true;
    }
  }
  *starts = __ballot(start);
  *wrong = __ballot(bad);
  *lives = __ballot(live);
}
// Rows of the piece that starts at bit r.
__device__ __forceinline__ int piece_len(unsigned long long starts, unsigned long long lives, int r) {
  const unsigned long long later = r == 63 ? 0ull : starts >> (r + 1);
  return later ? __builtin_ctzll(later) + 1 : __popcll(lives) - r;
}

}  // namespace rfmls
