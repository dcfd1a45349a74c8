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

// Which convolutions go row by row (a workgroup per row) and which by edge ranges.  V rows, E edges, `resident`: workgroups
// that the machine holds at once.
//
// Forward and second order: by rows, but for many rows of a few edges each, most of whose workgroup is idle.  (Rows without an
// edge cost little again.)  us, ranges -> rows.  Forward, 128 channels, 20 000 nodes: degree 0.1 82 -> 54, 0.5 84 -> 98, 1
// 96 -> 128, 2 130 -> 158, 4 210 -> 212, 7 328 -> 298; 9 000 nodes of degree 2 71 -> 69; 96 channels, 20 000 of
// degree 4 83 -> 90; 32 channels fp64, 20 000 of degree 2 80 -> 110, 9 000 52 -> 43.
// Second order, 128 channels (512 resident), 9 000 nodes: degree 1 162 -> 185, 3 339 -> 311; 20 000 of degree 0.1 160 -> 138, 0.25
// 169 -> 196, 2 560 -> 535; 5 000 of degree 1 101 -> 103, 7 000 134 -> 149; 96 channels (768) 9 000 of degree 1 76 -> 54, 20 000 125 -> 139,
// of degree 2 189 -> 180.  Where workers share waves, 32 channels (1 024), 20 000 nodes: degree 2 163 -> 190, 3 212 -> 220, 4 269 -> 266;
// 12 000 of degree 1 79 -> 77.
inline bool forward_by_rows(int64_t V, int64_t E) { return V <= 10000 || E / 5 >= V || E <= V / 8; }
inline bool double_by_rows(int64_t V, int64_t E, int64_t resident, int spw) {
  return V <= 12 * resident || E / (spw > 1 ? 4 : 2) >= V || E <= V / 8;
}

// The backward, whose weights come in the order of the senders: 0 by ranges, 1 by rows, 2 by rows with non-temporal streams.
//  - Where several workers' weights share a cache line (`few_channels`: 4 channels, 20 000 nodes of degree 32, 178 -> 97 us; degree
//    0.5 22 -> 16): rows.
//  - For short streams: one launch instead of three.  The limit is where the last workgroups leave the machine idle for as long:
//    64 channels fp64, 1 500 nodes of degree 36, 104 us by ranges, 112 by rows; where workers share waves, 32 channels, 3 000
//    nodes of degree 18, 77 and 66, of degree 36, 134 and 135, 9 000 of degree 7 94 and 103; with more than 128 registers, so one
//    workgroup of eight waves a CU, 32 channels fp64, 800 of degree 18, 52 and 44, of degree 36, 81 and 87; 128 channels, 300 of
//    degree 9, 31 and 28, of degree 18, 38 and 40.
//    Rows of fewer than six edges leave waves idle: by rows only as many of them as the launches cost.  128 channels (256
//    resident), 400 nodes of degree 3 27 -> 23, 800 32 -> 36, of degree 1 20 -> 26; 32 channels fp64 (512), 800 of degree 1 20 -> 18,
//    1 500 21 -> 26, 5 000 of degree 3 60 -> 76; 96 channels (512), 1 500 of degree 1 18 -> 18.5, 5 000 32 -> 40, 9 000 of degree 4
//    77 -> 93, but 3 300 of degree 6 48 -> 45; 32 channels (1 024), 5 000 of degree 1 32 -> 30, 9 000 39 -> 45.
//  - For many rows, when the workgroups of fewer waves come in three rounds or more: 96 channels fp64, 5 000 nodes of
//    degree 9, 138 -> 129, fp32 3 000 of degree 36 160 and 162, 5 000 255 and 250; 128 channels, 3 000 of degree 18, 227 -> 224
//    (2 000 of degree 32 261 -> 266).  One fp64 channel a lane needs four rounds and rows worth the workgroup: 32 channels, 5 000 of degree
//    36, 396 -> 409, 12 000 931 -> 912; 48 channels, 20 000 of degree 9, 273 -> 293, of degree 36, 1029 -> 1013.  The others six edges a
//    row: 128 channels, 20 000 nodes of degree 1 132 -> 182, 4 374 -> 380, 7 598 -> 594.
struct BackwardRows {
  bool few_channels, f64;
  int cpl, spw;                          // channels per lane, workers per wave
  bool many_registers;                   // more than 128
  int64_t resident, resident_nt;         // of the plain and of the non-temporal kernel
};
inline int backward_by_rows(const BackwardRows& k, int64_t V, int64_t E, int64_t stream_bytes) {
  const int64_t mb = (int64_t)1 << 20;
  if (k.few_channels) return stream_bytes > 256 * mb ? 2 : 1;
  const int64_t few = k.many_registers ? (k.cpl > 1 ? 40 : 72) : k.spw > 1 ? 120 : 96;
  const bool filled = E / 6 >= V;
  if (stream_bytes <= few * mb) return filled || V <= (k.many_registers ? 2 : k.spw > 1 ? 5 : 3) * k.resident;
  const bool many = k.f64 && k.cpl == 1 ? V >= 4 * k.resident_nt && E / 16 >= V : V >= 3 * k.resident_nt && filled;
  return many ? 2 : 0;
}

}  // namespace cgtp
