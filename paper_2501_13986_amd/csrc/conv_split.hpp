// How a convolution cuts its edges, and how many pieces of cut rows that can leave: plain arithmetic on sizes, shared by the
// launches and the workspace, so that the workspace never falls with the number of edges (a call on a smaller graph must
// neither free a buffer that a captured one still uses nor allocate inside a capture).
#pragma once

#include <algorithm>
#include <cstdint>
#include <initializer_list>

namespace cgtp {

// Edge ranges of a convolution kernel: one per resident worker (`all` of them), but where that leaves fewer than two edges
// each, ranges of three (of eight for workers that share a wave with many others), as long as 1 024 waves have work: every
// range costs a row search and up to two pieces of split rows for the merge kernel.
// forward + backward, one edge range per worker -> this: 3 000 nodes of 4 channels 136 -> 69 us, 300 nodes of 96 channels
// 46 -> 39, 300 nodes of 128 channels 69 -> 67 (second order 93 -> 85).  With two edges per worker already, three are
// slower (second order, 700 nodes of 32 channels 72 -> 76), and so is a range of four for each of fewer than 1 024 waves
// (27 nodes of 32 channels 26 -> 30).
inline int64_t conv_ranges(int64_t all, int spw, int64_t E) {
  const int64_t few = spw >= 8 ? 8 : 3;
  if (E >= 2 * all) return all;
  return std::min(std::min(E, all), std::max<int64_t>(1024 * spw, E / few));
}

// Rows of more than 2^lg edges are cut into windows of that size: 16 edges for each worker of a row, and no more than 1 024
// windows, nor than leave the pieces (two rows of `row_bytes` a window) within the static array of conv_forward_static, so
// that it cuts as conv_forward does.
constexpr int64_t kRowWindows = 1024;
constexpr int64_t kRowPieceBytes = (int64_t)32 << 20;
inline int64_t row_windows(int lg, int64_t E) { return ((E - 1) >> lg) + 1; }
inline int row_lg(int64_t workers, int64_t E, int64_t row_bytes) {
  int lg = 0;
  while (((int64_t)1 << lg) < 16 * workers || row_windows(lg, E) > kRowWindows || row_windows(lg, E) * 2 * row_bytes > kRowPieceBytes) ++lg;
  return lg;
}
// The windows of row_lg halve whenever their size doubles; this is the most that any graph of up to E edges has.
inline int64_t most_row_windows(int64_t workers, int64_t E, int64_t row_bytes) {
  return std::min(row_windows(row_lg(workers, 1, row_bytes), E), std::min(kRowWindows, kRowPieceBytes / (2 * row_bytes)));
}

// The most pieces of cut rows (two a range, two a window) that any graph of up to E edges leaves, walked by ranges or by one of
// the row kernels (workers of a row; 0: the plan has no such kernel).
inline int64_t most_pieces(int64_t all, int spw, std::initializer_list<int64_t> row_workers, int64_t E, int64_t row_bytes) {
  int64_t most = conv_ranges(all, spw, E);
  for (int64_t workers : row_workers)
    if (workers) most = std::max(most, most_row_windows(workers, E, row_bytes));
  return 2 * most;
}

}  // namespace cgtp
