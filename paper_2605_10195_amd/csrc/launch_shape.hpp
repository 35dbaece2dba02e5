// Launch shapes that follow from sizes alone, apart from the kernels so that they can be checked without a GPU.
#pragma once

#include <algorithm>
#include <cstdint>

namespace spex {

// Forms of the split path's launch of all items (MFMA-tiled pools); what they are stands at spex_split_attn_kernel.
enum SplitForm : int32_t { kSplitFull, kSplitLean, kSplitTiles };
// Workgroups a compute unit.
constexpr int split_occupancy(int head_dim, SplitForm form) {
  return head_dim == 64 ? (form == kSplitLean ? 5 : 3) : (form == kSplitLean ? 3 : 2);
}

// Most workgroups of a launch whose items of many rows go as row tiles of 16 nt, a workgroup each; `pages` is the mean length of the
// tiles' items.  512 run at once, two a compute unit.  Through LDS / as tiles, us: a prompt of 4096 under 16
// rows bf16 12.2 / 9.5, fp8 13.9 / 10.5, prompts under 48 to 128 rows 14.6 / 10.3, 24.3 / 18.7; of 513 to 1024 tiles
// 14.5 / 12.7, 13.1 / 13.3, 14.2 / 17.7; of more 15.7 / 18.9, 22.7 / 28.2.  bf16 heads of 64 gain too little beyond:
// 544 13.3 / 11.7, 1536 33 / 24, 1408 28 / 31, 2176 20.3 / 20.5, 3072 35 / 44.
// fp8, one set of 16 rows: up to four rounds where the items are long, because the items through LDS take as long a block
// whatever its bytes; every round costs the tiles some 3 us however short they are.  Heads of 128, prompts of 2000 tokens and more:
// 1344 workgroups 41 / 25, 1728 34 / 26, 2016 43 / 35, 1280 27 / 23, 1920 33 / 31, 2560 35 / 42, 4480 50 / 57; nodes of 1 page: 1920
// 13.3 / 17.6, of 2 pages 1344 13.0 / 15.8.  Heads of 64, items of 4 pages: 1728 12.2 / 14.4, 1664 10.1 / 12.0, of 8 13.3 / 14.6,
// 12.4 / 11.9, of 24 21.2 / 17.1, 22.7 / 15.8, of 64 44.0 / 24.0, 46.9 / 25.4.
// Over 3891 drawn requests, not those of the fit, the choice takes 0.90 of the time through LDS, 65 of them are slower so by 2 to
// 12 %; with 2048 whatever the length 192 of 2325 are, by up to 31 %.
constexpr int64_t most_row_tiles(bool fp8, int32_t nt, int32_t head_dim, int64_t pages) {
  return fp8 && nt == 1 ? std::clamp<int64_t>(head_dim == 64 ? 512 + 160 * pages : 384 + 96 * pages, 512, 2048) : 512;
}

struct SplitSizes {
  int32_t head_dim;
  bool fp8;
  int32_t nt;                      // sets of 16 rows of the longest private item's kind: 1 or 2
  int64_t wide, shared, streamed;  // items of up to 128 rows, of up to 64, and those of up to 16 with the private ones
  int64_t tiles, tile_pages;       // row tiles of the first two, pages of all of these together
  int32_t longest;                 // pages of the longest of the others
};
inline SplitForm split_form(const SplitSizes &s) {
  if (s.tiles > 0 && s.tiles + s.streamed <= most_row_tiles(s.fp8, s.nt, s.head_dim, s.tile_pages / s.tiles)) return kSplitTiles;
  // More workgroups than run at a time in the other form, and no long items, which want their loads a block ahead.
  // bf16 heads of 128 read as fast with two workgroups a compute unit.  Times of both forms, us: fp8 heads of 128, items of 8
  // pages, 6144 workgroups 73.6 / 63.6, 1536 25.0 / 22.7, of 16 pages 768 18.5 / 16.4, of 128 pages 768 36.4 / 37.2;
  // heads of 64, 8 pages, 1536 23.3 / 21.2 (fp8 24.9 / 20.4); bf16 heads of 128, 16 pages, 3072 82.6 / 85.1.
  if (s.nt == 1 && (s.fp8 || s.head_dim == 64) && s.wide == 0 && s.shared + s.streamed > 256 * split_occupancy(s.head_dim, kSplitFull) &&
      s.longest <= 16)
    return kSplitLean;
  return kSplitFull;
}

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
  // kv heads before query tokens in the grid, so that the workgroups of a query token, which read neighbouring rows, run at the same
  // time (and a kv head's on the XCDs that had its items where they are a multiple of 4).  The attention launch gains as well
  // as the merge.  Query tokens first / kv heads first, us a call, medians of 5 to 7 runs: heads 16/4/128 26.8 / 24.8, 15.0 / 14.0,
  // 22.4 / 19.6, 28/4/128 20.5 / 19.2, 33.5 / 32.0, 16/2/64 15.9 / 14.7, 17.4 / 16.6, 14/2/128 23.1 / 21.9, 24/6/128 34.9 / 33.8,
  // 27.0 / 25.7, 12/3/128 18.8 / 18.0; the other way round 24 trees of 8 branches, 8/2/128 12.3 / 13.1, 16/2/64 11.5 / 12.3, and
  // 24/6/128 20.2 / 21.0.  One kv head: 26.9 / 27.3, 22.9 / 24.5 with its parts first.
  s.heads_first = num_kv_heads > 1 && n_qtok <= 65535;
  return s;
}

}  // namespace spex
