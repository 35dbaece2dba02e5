// Host-only checks of the planner's automatic choices, built with sanitizers by test_host_sanitizers.py:
// a plan that length patches bring up to date keeps the kernels that a fresh plan of the same request
// would get, and the rules hold at their boundaries.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "../paper_2605_10195_amd/csrc/launch_shape.hpp"
#include "../paper_2605_10195_amd/csrc/planner.hpp"

using namespace spex;

static int failures = 0;
#define CHECK(cond, ...) \
  do { \
    if (!(cond)) { std::printf("line %d: " #cond " ", __LINE__); std::printf(__VA_ARGS__); std::printf("\n"); ++failures; } \
  } while (0)

struct Forest {
  PageTable pt;
  std::vector<int32_t> leaves, q_lens;
  Forest(int64_t pages, int page_size) : pt(pages, page_size, nullptr) {}
  // `roots` prompts with `branches` nodes each below them (0: the prompts themselves are asked for)
  void add(int roots, int prompt, int branches, int tokens, int q_len = 1) {
    const int r = pt.fork(kNoNode, roots);
    for (int i = 0; i < roots; ++i) {
      pt.append(r + i, prompt, nullptr);
      if (branches == 0) ask(r + i, q_len);
    }
    for (int i = 0; i < roots && branches > 0; ++i) {
      const int f = pt.fork(r + i, branches);
      for (int k = 0; k < branches; ++k) {
        pt.append(f + k, tokens, nullptr);
        ask(f + k, q_len);
      }
    }
  }
  void ask(int u, int q_len) {
    leaves.push_back(u);
    q_lens.push_back(q_len);
  }
};

struct Made {
  Planner planner;
  Plan plan;
  Made(const Forest &f, int Hq, int Hkv, int prefix_chunk = 0, int suffix_chunk = 0) {
    planner.pool = {f.pt.page_size() == 16, f.pt.page_size() < 4, 128, 2};
    const PlanError e = planner.begin(f.pt, f.leaves.data(), f.q_lens.data(), nullptr, static_cast<int32_t>(f.leaves.size()), Hq,
                                      Hkv, prefix_chunk, suffix_chunk, 0, 0, &plan);
    CHECK(e == PlanError::kOk, "begin");
  }
};

// Branches that grow a token each per round: as long as the patches hold, choice and halves are those
// of a plan made afresh.
static void growth(int roots, int prompt, int branches, int tokens, int Hq, int Hkv, int rounds) {
  Forest f(roots * (prompt / 16 + 2 + branches * ((tokens + rounds) / 16 + 2)), 16);
  f.add(roots, prompt, branches, tokens);
  Made m(f, Hq, Hkv);
  const bool first = m.planner.prefers_walk(f.pt, &m.plan);
  std::vector<int32_t> patches;
  int patched = 0;
  for (int t = 0; t < rounds; ++t) {
    for (int32_t u : f.leaves) f.pt.append(u, 1, nullptr);
    patches.clear();
    if (!m.planner.patch_lengths(f.pt, &m.plan, &patches)) break;
    ++patched;
    Made fresh(f, Hq, Hkv);
    const bool now = m.planner.prefers_walk(f.pt, &m.plan), want = fresh.planner.prefers_walk(f.pt, &fresh.plan);
    CHECK(now == first, "%d roots of %d, %d branches: the choice changed after %d tokens", roots, prompt, branches, t + 1);
    CHECK(now == want, "%d roots of %d, %d branches: a fresh plan chooses otherwise after %d tokens", roots, prompt, branches, t + 1);
    if (first) CHECK(m.plan.walk_halves == fresh.plan.walk_halves, "halves after %d tokens", t + 1);
  }
  CHECK(patched >= std::min(rounds, first ? 40 : 1), "only %d rounds patched", patched);
}

int main() {
  growth(8, 2500, 24, 17, 32, 8, 64);
  growth(8, 3000, 32, 17, 32, 8, 64);
  growth(32, 600, 16, 40, 32, 8, 64);
  growth(40, 700, 8, 20, 16, 4, 64);

  // one branch a tree and one kv head: a workgroup per tree
  auto halves = [](int even, int longer) {
    Forest f(even * 4 + 4000, 16);
    f.add(even, 64, 0, 0);
    if (longer) f.add(1, 16 * 60, 0, 0);
    Made m(f, 4, 1);
    m.planner.ensure_walk(f.pt, &m.plan);
    CHECK(m.plan.walk_ok && m.plan.walk_real_items == even + (longer ? 1 : 0), "%d workgroups", m.plan.walk_real_items);
    return m.plan.walk_halves;
  };
  CHECK(halves(256, 0), "256 even workgroups");
  CHECK(!halves(257, 0), "257 even workgroups");
  CHECK(halves(447, 1), "448 workgroups, one of them long");
  CHECK(!halves(448, 1), "449 workgroups");
  // equal workgroups of many 16 KiB blocks; 32 and 33 row blocks a root; a ragged launch of short paths
  auto halves_of = [](int roots, int prompt, int branches, int longer, int Hq, int Hkv, int kv_bytes, int row_tiles = 0) {
    Forest f(static_cast<int64_t>(roots) * (prompt / 16 + 2 + branches) + longer + 16, 16);
    f.add(roots, prompt, branches, 16);
    if (longer) f.add(1, 16 * longer, 0, 0);
    Made m(f, Hq, Hkv);
    m.planner.pool = {true, false, 128, kv_bytes};
    CHECK(m.planner.begin(f.pt, f.leaves.data(), f.q_lens.data(), nullptr, static_cast<int32_t>(f.leaves.size()), Hq, Hkv, 0, 0, row_tiles, 0,
                          &m.plan) == PlanError::kOk, "begin");
    m.planner.ensure_walk(f.pt, &m.plan);
    return m.plan.walk_halves;
  };
  CHECK(halves_of(240, 3200, 0, 0, 4, 1, 2), "24000 blocks of 16 KiB");
  CHECK(!halves_of(240, 3240, 0, 0, 4, 1, 2), "24480 blocks of 16 KiB");
  CHECK(halves_of(240, 3240, 0, 0, 4, 1, 1) && halves_of(240, 3240, 0, 0, 4, 1, 2, 2), "24480 blocks of 8 KiB, or with two row tiles");
  CHECK(halves_of(120, 6480, 2, 0, 4, 1, 2), "24840 blocks of 16 KiB, two branches a root");
  CHECK(halves_of(3, 600, 4 * 32, 0, 32, 2, 2, 1) && !halves_of(3, 600, 4 * 33, 0, 32, 2, 2, 1), "three roots on four pairs of XCDs");
  CHECK(halves_of(300, 20, 0, 32, 4, 1, 2) && !halves_of(300, 20, 0, 30, 4, 1, 2), "longest of 16 and of 15 blocks");

  // no estimate beyond 512 workgroups or 1024 query tokens: the tree-walk kernel
  auto choice = [](int trees, int tokens, int q_len) {
    Forest f(trees * (tokens / 16 + 1), 16);
    f.add(trees, tokens, 0, 0, q_len);
    Made m(f, 4, 1);
    m.planner.pool.head_dim = 64;
    return m.planner.prefers_walk(f.pt, &m.plan);
  };
  CHECK(!choice(512, 20000, 1), "512 workgroups on long paths");
  CHECK(choice(513, 20000, 1), "513 workgroups");
  CHECK(!choice(341, 16000, 3), "1023 query tokens");
  CHECK(choice(342, 16000, 3), "1026 query tokens");
  CHECK(!choice(16, 20000, 1), "few long paths");
  CHECK(choice(16, 512, 1), "few short paths");

  // pools of the generic kernel: four times as many shared items of a long prompt
  for (bool generic : {false, true}) {
    Forest f(2000, 16);
    f.add(1, 16 * 1024, 4, 16);
    Made m(f, 8, 4);
    m.planner.pool = {false, generic, 40, 1};
    CHECK(m.planner.ensure_split(f.pt, &m.plan) == PlanError::kOk, "split lists");
    CHECK(m.plan.prefix_chunk_pages == (generic ? 8 : 16), "items of %d pages", m.plan.prefix_chunk_pages);
  }

  // automatic items, by page size: never more partial rows than the shortest items give, and items of
  // at least those lengths where the partial rows would be too many
  for (int P = 1; P <= 64; P *= 2)
    for (int q_len : {1, 64}) {
      Forest f(2048 / P + 32 * (128 / P + 1) + 1, P);
      f.add(1, 2048, 32, 128, q_len);
      const int lo_shared = P < 4 ? 16 : 128 / P, lo_private = P < 4 ? 8 : 128 / P;
      Made a(f, 32, 8), s(f, 32, 8, lo_shared, lo_private);
      CHECK(a.planner.ensure_split(f.pt, &a.plan) == PlanError::kOk, "split lists");
      CHECK(s.planner.ensure_split(f.pt, &s.plan) == PlanError::kOk, "split lists");
      CHECK(a.plan.n_partial_rows <= s.plan.n_partial_rows, "pages of %d, %d queries: %ld partial rows, %ld with the shortest items", P,
            q_len, static_cast<long>(a.plan.n_partial_rows), static_cast<long>(s.plan.n_partial_rows));
      CHECK(a.plan.prefix_chunk_pages >= lo_shared && a.plan.suffix_chunk_pages >= lo_private, "pages of %d, %d queries: items of %d and %d pages",
            P, q_len, a.plan.prefix_chunk_pages, a.plan.suffix_chunk_pages);
      if (s.plan.n_partial_rows > 40960)
        CHECK(a.plan.prefix_chunk_pages >= 16 && a.plan.suffix_chunk_pages >= 8, "pages of %d, %d queries: items of %d and %d pages", P, q_len,
              a.plan.prefix_chunk_pages, a.plan.suffix_chunk_pages);
    }

  // row tiles one by one: 6 rows a branch, 27 branches, prompts of `prompt` tokens
  auto by_tile = [](int prompt, int row_tiles, int waves, int kv_bytes) {
    Forest f(400, 16);
    f.add(1, prompt, 27, 70);
    Made m(f, 6, 1);
    m.planner.pool = {true, false, 128, kv_bytes};
    CHECK(m.planner.begin(f.pt, f.leaves.data(), f.q_lens.data(), nullptr, 27, 6, 1, 0, 0, row_tiles, waves, &m.plan) == PlanError::kOk, "begin");
    m.planner.ensure_walk(f.pt, &m.plan);
    const bool few = m.plan.walk_tiles_touched * (row_tiles == 4 ? 4 : 5) < m.plan.walk_tiles_held * (row_tiles == 4 ? 3 : 4);
    CHECK(few == (prompt < 1000 && row_tiles > 1), "prompt %d, %d tiles: %ld of %ld touched", prompt, row_tiles, static_cast<long>(m.plan.walk_tiles_touched),
          static_cast<long>(m.plan.walk_tiles_held));
    return m.plan.walk_by_tile;
  };
  CHECK(by_tile(40, 2, 4, 1) && by_tile(40, 2, 8, 1) && by_tile(40, 4, 4, 1) && by_tile(40, 4, 4, 2), "short prompt");
  CHECK(!by_tile(40, 2, 4, 2) && !by_tile(40, 1, 4, 1) && !by_tile(40, 2, 2, 1), "bf16 with two tiles, one tile, path split in two");
  CHECK(!by_tile(5000, 2, 4, 1) && !by_tile(5000, 4, 4, 2), "long prompt");

  // the split path's launches, one or in phases: (roots, branches, queries, heads) -> workgroups at the bound
  auto phases = [](int roots, int branches, int q_len, int Hq, int Hkv, int dim, bool tiled = true) {
    Forest f(roots * (3 + 2 * branches), 16);
    f.add(roots, 40, branches, 20, q_len);
    Made m(f, Hq, Hkv);
    m.planner.pool = {tiled, false, dim, 2};
    CHECK(m.planner.ensure_split(f.pt, &m.plan) == PlanError::kOk, "split lists");
    return m.plan.split_phases;
  };
  CHECK(!phases(256, 1, 1, 40, 2, 128), "512 private items of 20 rows");
  CHECK(phases(257, 1, 1, 40, 2, 128), "514 private items of 20 rows");
  CHECK(!phases(34, 4, 1, 71, 1, 64), "34 * (4 * 3 + 3) = 510 workgroups");
  CHECK(phases(35, 4, 1, 71, 1, 64), "525 workgroups");
  CHECK(!phases(512, 16, 1, 8, 2, 128), "16384 private items of 4 rows");
  CHECK(phases(513, 16, 1, 8, 2, 128), "16416 private items of 4 rows");
  CHECK(!phases(64, 16, 1, 16, 4, 64), "4096 private items of 4 rows, head dim 64");
  CHECK(phases(65, 16, 1, 16, 4, 64), "4160 private items of 4 rows, head dim 64");
  CHECK(!phases(513, 16, 1, 8, 2, 128, false), "row-major");

  // items of more than 16 rows cut for phases that go in one launch all the same
  auto together = [](int roots, int branches, int q_len, int Hq, int Hkv, int dim, int prompt = 40) {
    Forest f(roots * (3 + prompt / 16 + 2 * branches), 16);
    f.add(roots, prompt, branches, 20, q_len);
    Made m(f, Hq, Hkv);
    m.planner.pool = {true, false, dim, 2};
    CHECK(m.planner.ensure_split(f.pt, &m.plan) == PlanError::kOk, "split lists");
    return m.plan.split_together;
  };
  CHECK(!together(256, 1, 1, 40, 2, 128) && together(257, 1, 1, 40, 2, 128), "512 items are not cut for phases, 514 are");
  CHECK(together(768, 1, 1, 40, 2, 128) && !together(769, 1, 1, 40, 2, 128), "1536 and 1538 items");
  CHECK(together(68, 4, 1, 71, 1, 64) && !together(69, 4, 1, 71, 1, 64), "1020 and 1035 workgroups, head dim 64");
  CHECK(together(13, 8, 8, 32, 8, 128, 600) && !together(14, 8, 8, 32, 8, 128, 600), "1456 and 1568 workgroups, prompts of 38 pages");
  CHECK(!together(513, 16, 1, 8, 2, 128), "4 rows");

  // pieces' records at a stride: pairs a query token, 0 where nothing is merged (every row in one piece) or where they
  // would take more room
  auto stride = [](int roots, int prompt, int branches, int more) {
    Forest f(2 * roots * (2 + prompt / 16 + branches * 2) + more / 16 + 1, 16);
    f.add(roots, prompt, branches, 20);
    if (more > 0) f.add(1, more, 0, 0);
    Made m(f, 8, 2, 1, 1);
    CHECK(m.planner.ensure_split(f.pt, &m.plan) == PlanError::kOk, "split lists");
    CHECK(static_cast<int>(m.plan.merge_rec.size()) == 2 * m.plan.merge_stride * static_cast<int>(f.leaves.size()), "%d roots", roots);
    for (size_t t = 0; t < f.leaves.size() && m.plan.merge_stride > 0; ++t)
      for (int k = 0; k < m.plan.merge_stride; ++k) {
        const int e = m.plan.part_indptr[t] + k;
        const bool there = e < m.plan.part_indptr[t + 1];
        const int32_t *rec = &m.plan.merge_rec[2 * (t * m.plan.merge_stride + k)];
        CHECK(rec[0] == (there ? m.plan.part_base[e] : -1) && (!there || rec[1] == m.plan.part_hstride[e]), "%d roots", roots);
      }
    return m.plan.merge_stride;
  };
  CHECK(stride(3, 40, 4, 0) == 5 && stride(20, 40, 4, 33) == 5, "prompts of 3 pages, branches of 2, a prompt alone of 3");
  CHECK(stride(3, 40, 4, 400) == 0, "a prompt alone of 25 pages");
  CHECK(stride(5, 16, 0, 0) == 0, "one piece each");

  // shared items cut to go as row tiles of 16: pages of an item, 0 if they are not
  auto tiles = [](int roots, int prompt, int branches, int dim, int kv_bytes, int chunk = 0) {
    Forest f(roots * (1 + (prompt + 15) / 16 + 2 * branches), 16);
    f.add(roots, prompt, branches, 20);
    Made m(f, 32, 8, chunk), bf16(f, 32, 8, chunk);
    m.planner.pool = {true, false, dim, kv_bytes};
    CHECK(m.planner.ensure_split(f.pt, &m.plan) == PlanError::kOk, "split lists");
    CHECK(bf16.planner.ensure_split(f.pt, &bf16.plan) == PlanError::kOk, "split lists");
    CHECK(!bf16.plan.split_tiles, "bf16 heads of 128");
    CHECK(m.plan.n_partial_rows <= bf16.plan.n_partial_rows, "%d prompts of %d: more partial rows", roots, prompt);
    return m.plan.split_tiles ? m.plan.prefix_chunk_pages : 0;
  };
  CHECK(tiles(2, 6000, 8, 128, 1) == 32, "128 private items leave 192 of two tiles for 6000 pages and heads");
  CHECK(tiles(2, 6000, 16, 64, 1) == 47, "256 private items leave 128 of four tiles, heads of 64");
  CHECK(tiles(2, 6000, 32, 128, 1) == 94 && tiles(2, 6000, 32, 128, 2) == 0 && tiles(2, 6000, 8, 64, 2) == 0, "no room: 64 items; bf16");
  CHECK(tiles(2, 300, 5, 64, 1) == 8, "short prompts: items of 8 pages");
  CHECK(tiles(2, 6000, 4, 128, 1) == 0 && tiles(2, 6000, 5, 128, 1) > 0, "16 and 20 rows");
  CHECK(tiles(2, 6000, 8, 128, 1, 24) == 0, "length given");
  CHECK(tiles(12, 2000, 16, 128, 1) == 188 && tiles(13, 2000, 16, 128, 1) == 0, "1920 and 2080 tiles");

  // form of the one launch; `pages` of a prompt of `items` of them a branch
  auto form = [](int roots, int items, int pages, int branches, int Hq, int Hkv, int dim, int kv_bytes, int tokens = 20) {
    Forest f(roots * (items * pages + 2 * branches * (1 + tokens / 16)), 16);
    f.add(roots, 16 * items * pages, branches, tokens);
    Made m(f, Hq, Hkv, pages);
    m.planner.pool = {true, false, dim, kv_bytes};
    CHECK(m.planner.ensure_split(f.pt, &m.plan) == PlanError::kOk, "split lists");
    return m.plan.split_form;
  };
  CHECK(form(24, 5, 24, 16, 8, 2, 64, 1) == kSplitTiles && form(24, 7, 24, 16, 8, 2, 64, 1) != kSplitTiles, "1728 and 2112 workgroups");
  CHECK(form(4, 6, 24, 24, 32, 8, 128, 1) == kSplitTiles && form(4, 7, 24, 24, 32, 8, 128, 1) != kSplitTiles, "1920 and 2112");
  CHECK(form(24, 2, 4, 16, 8, 2, 64, 1) == kSplitTiles && form(24, 3, 4, 16, 8, 2, 64, 1) != kSplitTiles, "1152 of 4 pages and 1344");
  CHECK(form(4, 5, 8, 24, 32, 8, 64, 1) == kSplitTiles && form(4, 6, 8, 24, 32, 8, 64, 1) != kSplitTiles, "1728 of 8 pages and 1920");
  CHECK(form(4, 3, 10, 24, 32, 8, 128, 1) == kSplitTiles && form(4, 4, 10, 24, 32, 8, 128, 1) != kSplitTiles, "1344 of 10 pages and 1536");
  CHECK(form(8, 1, 1, 16, 8, 2, 128, 1) == kSplitTiles && form(16, 1, 1, 16, 8, 2, 128, 1) == kSplitLean, "320 of a page and 640");
  CHECK(form(6, 4, 24, 16, 8, 2, 128, 2) == kSplitTiles && form(6, 7, 24, 16, 8, 2, 128, 2) == kSplitFull, "bf16: 384 and 528");
  CHECK(form(6, 4, 24, 16, 8, 2, 64, 2) == kSplitTiles && form(6, 7, 24, 16, 8, 2, 64, 2) == kSplitFull, "bf16: 384 and 528");

  // row tiles are those that items have, whatever the largest group of the request, and a list's span is its own largest item's
  auto mixed = [](int small, int wide_branches, int *span) {
    Forest f(small * 20 + 200, 16);
    f.add(small, 60, 5, 20);
    if (wide_branches > 0) f.add(1, 60, wide_branches, 20);
    Made m(f, 8, 2);
    m.planner.pool = {true, false, 128, 2};
    CHECK(m.planner.ensure_split(f.pt, &m.plan) == PlanError::kOk, "split lists");
    span[0] = m.plan.coop_span[0];
    span[1] = m.plan.coop_span[1];
    return m.plan.split_form;
  };
  int span[2];
  CHECK(mixed(36, 0, span) == kSplitTiles && span[0] == 20 && span[1] == 1, "504 workgroups");
  CHECK(mixed(33, 16, span) == kSplitTiles && span[0] == 64, "132 tiles of 20 rows, 8 of 64 and 362 private items");
  CHECK(mixed(30, 33, span) == kSplitTiles && span[0] == 20 && span[1] == 128, "one group of 132 rows");
  CHECK(mixed(37, 0, span) == kSplitFull, "518 workgroups");

  // requests of more rows than a row block holds (two tiles of 16 a wavefront, four wavefronts) have their block lists cut
  auto cut = [](int q_len, int Hq, int Hkv) {
    Forest f(200, 16);
    f.add(2, 300, 2, 150, q_len);
    Made m(f, Hq, Hkv);
    m.planner.ensure_walk(f.pt, &m.plan);
    CHECK(m.plan.walk_ok && m.plan.walk_row_tiles == 2 && m.plan.walk_waves == 4, "two tiles, four wavefronts");
    return m.plan.walk_cut;
  };
  CHECK(!cut(32, 8, 2) && cut(33, 8, 2), "128 and 132 rows");

  // merge workgroups: within 256 threads, every row in one of them, at least half full wherever there are rows enough, the heads of
  // a kv head in equal shares, and no grid dimension but the first beyond 65535
  for (int Hkv : {1, 3, 4, 32})
    for (int G : {1, 2, 3, 4, 7, 8, 20, 71})
      for (int D : {1, 30, 40, 64, 96, 128, 255, 256})
        for (int64_t n : {1, 7, 512, 70000})
          for (int pieces : {2, 6, 40}) {
            const MergeShape m = merge_shape(Hkv, G, D, n, pieces);
            CHECK(m.threads() <= kMergeThreads && m.dv * m.vec == D && m.rows >= 1 && m.tokens >= 1 && m.tokens <= n, "%d %d %d", G, D, pieces);
            CHECK(m.rows * m.parts >= G && m.rows * (m.parts - 1) < G && m.rows * m.parts - G < m.parts, "%d %d %d", G, D, pieces);
            CHECK(2 * m.threads() >= kMergeThreads || m.tokens == n, "%d heads a kv head of %d, %d pieces: %d threads", G, D, pieces,
                  m.threads());
            CHECK(m.heads_first == (Hkv > 1 && n <= 65535), "%d kv heads, %d query tokens", Hkv, static_cast<int>(n));
          }

  if (failures == 0) std::printf("ok\n");
  return failures != 0;
}
