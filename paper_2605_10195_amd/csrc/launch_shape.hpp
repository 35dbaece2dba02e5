// Launch shapes that follow from sizes alone, apart from the kernels so that they can be checked without a GPU.
#pragma once

#include <algorithm>
#include <cstdint>

namespace spex {

// Merge kernel: block (dv, tokens << slice_log2, rows), see spex_lse_merge_kernel.
struct MergeShape {
  int32_t vec;          // dims a thread
  int32_t dv;           // threads across a row
  int32_t slice_log2;   // log2 of the slices of a row's pieces
  int32_t rows;         // query heads of one kv head a workgroup
  int32_t tokens;       // query tokens a workgroup
  int32_t parts;        // workgroups for the query heads of one kv head
  bool heads_first;     // order of the workgroups
  int32_t threads() const { return dv * (tokens << slice_log2) * rows; }
};
constexpr int32_t kMergeBatch = 4;      // pieces a slice requests together
constexpr int32_t kMergeThreads = 256;  // most threads of a workgroup

inline MergeShape merge_shape(int32_t num_kv_heads, int32_t heads_per_kv, int32_t head_dim, int64_t n_qtok, int32_t avg_pieces) {
  MergeShape s{};
  s.vec = head_dim % 4 == 0 ? 4 : 1;
  s.dv = head_dim / s.vec;
  // One slice per kMergeBatch pieces of the average row, so that a slice runs one or two batches.
  while (s.slice_log2 < 3 && (s.dv << (s.slice_log2 + 1)) <= kMergeThreads && (kMergeBatch << s.slice_log2) < avg_pieces) ++s.slice_log2;
  const int32_t row = s.dv << s.slice_log2, room = kMergeThreads / row;
  // Query heads in equal shares: with 5 of them, 4 and 1 (heads 40/8/128, 650 query tokens of 24 pieces 15.7 us, 14.1 so; 72/8/128,
  // 1600 of 2 pieces 40.0 and 32.6).
  s.parts = (heads_per_kv + room - 1) / room;
  s.rows = (heads_per_kv + s.parts - 1) / s.parts;
  // Several query tokens where one leaves a workgroup fewer than half of its threads (figures at the kernel); with 128 threads
  // a second token costs more than it gives (32/8/128, 1 slice: 9.2 us, 9.6 with two).
  s.tokens = 2 * s.rows * row >= kMergeThreads ? 1 : static_cast<int32_t>(std::min<int64_t>(room / s.rows, n_qtok));
  // kv heads before query tokens in the grid where they are a multiple of 4: a kv head's workgroups then run on the one or two
  // XCDs that had its items.  Query tokens first / kv heads first, us a call, medians of 7 runs: heads 16/4/128 26.8 / 24.8,
  // 15.0 / 14.0, 22.4 / 19.6, 28/4/128 20.5 / 19.2, 33.5 / 32.0; with 2, 3 and 6 kv heads either may win: 8/2/128
  // 12.4 / 13.0, 18.8 / 18.7, 16/2/64 11.5 / 12.1, 16.9 / 16.4, 12/3/128 13.6 / 14.0, 18.6 / 18.2, 24/6/128 20.2 / 21.0, 34.7 / 33.8.
  s.heads_first = num_kv_heads % 4 == 0 && n_qtok <= 65535;
  return s;
}

}  // namespace spex
