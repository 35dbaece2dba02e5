// Launch interface between the C ABI layer and the HIP kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "launch_shape.hpp"

namespace spex {

enum Dtype : int32_t { kF32 = 0, kBF16 = 1, kFP8 = 2 };

// Element arrangement inside a (page, kv head) tile; see the pool layout in spex_tree.h.
enum Layout : int32_t { kRowMajor = 0, kMfmaTiled = 1 };

struct Shape {
  int32_t Hq, Hkv, G, D, P;
  int32_t q_dtype, kv_dtype, layout;
  int32_t page_tiles;  // tiles between the starts of consecutive pages inside a pool (>= Hkv)
};

// Everything the attention kernels read; all pointers DEVICE.
struct AttnArgs {
  const void *k_pool, *v_pool;
  const float *k_scale, *v_scale;
  const void *q;
  const int32_t *items;   // 8 ints per work item: {pg_begin, pg_count, qt_begin, qt_count, pbase,
                          //                       flags, kv_head, first_row}
  int32_t n_items;
  const int32_t *pg_rec;  // 2 ints per page entry: {page id, path position << 7 | valid tokens}
  const int32_t *qt_rec;  // 2 ints per row-set entry: {query token, visible path length}
  float *part_o;   // [partial rows][D] unnormalised sum of exp2(x - m) * V
  float *part_ml;  // [partial rows][2] = {m, l}: running maximum of x = score * log2(e), sum of exp2
  // every row of the launch has one piece only: write finished rows to out / lse instead (not the
  // generic kernel)
  bool finish;
  // rows of tasks flagged final, finished in place behind the launches of their other pieces: a row's
  // merge list (all entries but the last, which is the task itself)
  const int32_t *part_indptr, *part_base, *part_hstride;
  float *out, *lse;  // lse may be null
  float scale_log2;
  // Draft-tree visibility, or null for the causal chain: 2 ints per query token {index i of the
  // query in its request, mask}; with base = limit - 1 - i the query sees path positions below base
  // and position base + k iff bit k of the mask is set.
  const int32_t *qt_mask;
};

// Tree-walk kernel: one workgroup per work item.
struct WalkArgs {
  const void *k_pool, *v_pool;
  const float *k_scale, *v_scale;
  const void *q;
  const int32_t *items;   // 16 (2 or 4 wavefronts of rows per row block) or 32 (8) ints per workgroup: {kv head,
                          //   first block, shared blocks, private blocks of wavefronts 0..NW-1,
                          //   first qt_rec entry of each wavefront, qt_rec entries of each
                          //   wavefront, zeros.., row block}; no blocks = padding
  int32_t n_items;
  const int32_t *blocks;  // 8 ints per 32-token block: {page a, pos_a << 7 | valid_a, page b,
                          //   pos_b << 7 | valid_b (0: no page b), first row | (last row + 1) << 16
                          //   within the row block, flags (bit 0: token mask needed), 0, 0}
  const int32_t *qt_rec;  // 2 ints per row-set entry: {query token, visible path length}
  float *out, *lse;       // lse may be null
  float scale_log2;
  const int32_t *qt_mask; // as in AttnArgs; null for the causal chain
  bool cut;               // some request has more rows than a row block holds
};

struct MergeArgs {
  const int32_t *part_indptr, *part_base, *part_hstride;  // or, where stride > 0:
  const int32_t *rec;     // {base, hstride} of the query tokens' pieces, `stride` pairs each, base -1 behind the last one
  int32_t stride;
  const float *part_o, *part_ml;
  float *out, *lse;
  const int32_t *qt_ids;  // query tokens to merge, or null for 0 .. n_qtok-1
  int32_t n_qtok;         // number of query tokens handled by the launch
  int32_t avg_pieces;     // pieces of an average query token (a hint for the launch shape)
  bool heads_first;       // order of the workgroups and log2 of the slices of a row; set by launch_merge
  int32_t slice_log2;
};

// Page ids travel in the kernel arguments.  128 pages (2048 tokens of 16-token pages) per launch: with
// 512 the arguments of a short append cost 0.3 us more on the host (6.18 against 5.89 us a call).
constexpr int kMaxPagesPerScatter = 128;
struct ScatterArgs {
  void *k_pool, *v_pool;
  float *k_scale, *v_scale;              // pool scale arrays (fp8) or null
  const void *k_src, *v_src;             // [n_tokens][Hkv][D]
  const float *k_scale_src, *v_scale_src;  // [new pages][Hkv], already offset to this launch
  int32_t n_pages;                       // pages touched by this launch
  int32_t first_slot;                    // first written slot of page 0 (0 if it is new)
  int32_t n_tokens;                      // tokens written by this launch
  int32_t first_page_is_new;
  int32_t page_ids[kMaxPagesPerScatter];
};

// One token for each of n_nodes nodes in one launch.
struct AppendTokensArgs {
  void *k_pool, *v_pool;
  float *k_scale, *v_scale;                // pool scale arrays (fp8) or null
  const void *k_src, *v_src;               // [n_nodes][Hkv][D]
  const float *k_scale_src, *v_scale_src;  // [n_nodes][Hkv] (fp8; read only for nodes that start a page)
  const int32_t *dst;                      // 2 ints per node: {page id, slot | (page is new) << 8}; pinned host memory
  int32_t n_nodes;
  // fp8 pools only: k_src / v_src hold bf16 values, which the kernel encodes with the scale of the
  // page the token lands in (k_scale_src / v_scale_src for a page it starts)
  bool quantise;
  // Length patches of the cached plan, applied by the same launch (thread i < n_patches stores
  // patches[2 i + 1] into plan[patches[2 i]]); n_patches <= number of threads, 0 = none.
  int32_t *plan;
  const int32_t *patches;                  // pinned host memory, behind dst
  int32_t n_patches;
};

struct GatherArgs {
  const void *k_pool, *v_pool;
  const float *k_scale, *v_scale;
  void *k_out, *v_out;
  float *k_scale_out, *v_scale_out;
  int32_t n_pages, first_slot, n_tokens;
  int32_t page_ids[kMaxPagesPerScatter];
};

// Work items of the split path, by list: groups of more than 64 rows (spans of up to 128), of 17 to
// 64, of up to 16 rows, and private suffixes.  span: rows an item covers from its first row on.
struct ItemLists {
  const int32_t *items[4];
  int32_t n_items[4], span[4];
  SplitForm form;  // of launch_split on a tiled pool
};
bool has_mfma_kernel(const Shape &sh);
bool has_rowmajor_kernel(const Shape &sh, const AttnArgs &a);
// All lists in one launch; needs has_mfma_kernel or has_rowmajor_kernel.
hipError_t launch_split(const Shape &sh, const AttnArgs &a, const ItemLists &lists, hipStream_t stream);
// The same in up to four launches one behind the other, for launches with items enough (tiled pools).
hipError_t launch_split_phases(const Shape &sh, const AttnArgs &a, const ItemLists &lists, hipStream_t stream);
// a.items / a.n_items on the vector ALU; any shape.
hipError_t launch_generic_attention(const Shape &sh, const AttnArgs &a, int rows_per_item, hipStream_t stream);
hipError_t launch_merge(const Shape &sh, const MergeArgs &args, hipStream_t stream);
hipError_t launch_scatter(const Shape &sh, const ScatterArgs &a, hipStream_t stream);
// fp8 pools: k_src / v_src hold bf16 values; page scales are computed (started pages) or reused.
hipError_t launch_scatter_quantise(const Shape &sh, const ScatterArgs &a, hipStream_t stream);
hipError_t launch_gather(const Shape &sh, const GatherArgs &a, hipStream_t stream);
hipError_t launch_append_tokens(const Shape &sh, const AppendTokensArgs &a, hipStream_t stream);
// blob[pairs[2i]] = pairs[2i+1] for i < n (all DEVICE): patches the device copy of a plan.
hipError_t launch_patch(int32_t *blob, const int32_t *pairs, int32_t n, hipStream_t stream);
// Tree-walk kernel; ntw in {1, 2, 4} = 16-row tiles per wavefront and waves in {2, 4, 8} = wavefronts
// of rows per row block the lists were built for (2: run by four wavefronts, two on each set of
// rows, which split the path between them; ntw 1 or 2, no draft masks).
// halves (waves 4, ntw 1 or 2): eight wavefronts walk the lists made for four, two on each set of rows.
// by_tile: row tiles are worked on one by one, without those that a block does not touch.
hipError_t launch_tree_walk(const Shape &sh, const WalkArgs &a, int ntw, int waves, bool halves, bool by_tile,
                            hipStream_t stream);

}  // namespace spex
