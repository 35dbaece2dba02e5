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
  const int32_t room = kMergeThreads / (s.dv << s.slice_log2);
  s.rows = std::min(room, heads_per_kv);
  s.parts = (heads_per_kv + s.rows - 1) / s.rows;
  s.tokens = static_cast<int32_t>(std::min<int64_t>(room / s.rows, n_qtok));
  s.heads_first = num_kv_heads % 8 == 0 && n_qtok <= 65535;
  return s;
}

}  // namespace spex
