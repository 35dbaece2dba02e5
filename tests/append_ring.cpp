// The pinned lists of append_tokens, built by test_host_sanitizers.py from the library's own host sources over a HIP
// runtime that is made here: launches wait in queues and run only as far as the host waits for them, and each
// checks that its list still is what it was when it was launched.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <deque>
#include <map>
#include <vector>

#include "../include/spex_tree.h"
#include "../paper_2605_10195_amd/csrc/kernels.hpp"

static int failures = 0;
#define CHECK(ok, ...)                                                              \
  do {                                                                              \
    if (!(ok)) {                                                                    \
      std::printf("line %d: ", __LINE__), std::printf(__VA_ARGS__), std::printf("\n"); \
      ++failures;                                                                   \
    }                                                                               \
  } while (0)

struct Launch {
  const int32_t *list;
  std::vector<int32_t> then;
};
struct Queue {
  std::deque<Launch> waiting;
  long issued = 0, done = 0;
};
struct ihipEvent_t {
  int queue = -1;
  long upto = 0;
};

static std::map<int, Queue> queues;
static std::map<hipStream_t, int> queue_behind;  // which queue a handle stands for; a handle may be given out again
static int thread_now = 0, waits = 0, records_that_fail = 0;
static long overwritten = 0;
static std::map<const char *, size_t> pinned;

static int queue_of(hipStream_t s) { return s == hipStreamPerThread ? 1000 + thread_now : queue_behind[s]; }
static void run(Queue &q, long upto) {
  for (; q.done < upto; ++q.done) {
    const Launch &l = q.waiting.front();
    for (size_t i = 0; i < l.then.size(); ++i)
      if (l.list[i] != l.then[i]) {
        ++overwritten;
        break;
      }
    q.waiting.pop_front();
  }
}
static void run_all() {
  for (auto &q : queues) run(q.second, q.second.issued);
}

extern "C" {
const char *hipGetErrorString(hipError_t) { return "an error made by the test"; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { return *p = nullptr, hipErrorUnknown; }
hipError_t hipMalloc(void **p, size_t n) { return *p = std::malloc(n), hipSuccess; }
hipError_t hipFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  *p = std::malloc(n);
  pinned[static_cast<char *>(*p)] = n;
  return hipSuccess;
}
hipError_t hipHostFree(void *p) {
  const char *base = static_cast<char *>(p);
  for (auto &q : queues)
    for (const Launch &l : q.second.waiting) {
      const char *at = reinterpret_cast<const char *>(l.list);
      CHECK(at < base || at >= base + pinned[base], "pinned memory given back under a launch that reads it");
    }
  pinned.erase(base);
  std::free(p);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return run_all(), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  Queue &q = queues[queue_of(s)];
  return run(q, q.issued), hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return *e = new ihipEvent_t(), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return delete e, hipSuccess; }
hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { return hipErrorUnknown; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  if (records_that_fail > 0) return --records_that_fail, hipErrorUnknown;
  e->queue = queue_of(s);
  e->upto = queues[e->queue].issued;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  ++waits;
  return run(queues[e->queue], e->upto), hipSuccess;
}
}

namespace spex {
bool has_mfma_kernel(const Shape &) { return true; }
bool has_rowmajor_kernel(const Shape &, const AttnArgs &) { return false; }
hipError_t launch_split(const Shape &, const AttnArgs &, const ItemLists &, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_split_phases(const Shape &, const AttnArgs &, const ItemLists &, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_generic_attention(const Shape &, const AttnArgs &, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_merge(const Shape &, const MergeArgs &, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_scatter(const Shape &, const ScatterArgs &, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_scatter_quantise(const Shape &, const ScatterArgs &, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_gather(const Shape &, const GatherArgs &, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_patch(int32_t *, const int32_t *, int32_t, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_tree_walk(const Shape &, const WalkArgs &, int, int, bool, bool, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_append_tokens(const Shape &, const AppendTokensArgs &a, hipStream_t s) {
  Queue &q = queues[queue_of(s)];
  q.waiting.push_back({a.dst, std::vector<int32_t>(a.dst, a.dst + 2 * a.n_nodes)});
  ++q.issued;
  return hipSuccess;
}
}  // namespace spex

struct Tree {
  spex_tree_t *t = nullptr;
  std::vector<spex_node_t> nodes;
  char pool[16];
  explicit Tree(int n) : nodes(n) {
    spex_config_t c{};
    c.num_q_heads = c.num_kv_heads = 1;
    c.head_dim = 64;
    c.page_size = 16;
    c.q_dtype = c.kv_dtype = SPEX_BF16;
    c.num_pages = 200000;
    c.k_pool = c.v_pool = pool;
    CHECK(spex_tree_create(&c, &t) == SPEX_OK, "create");
    CHECK(spex_tree_fork(t, SPEX_NO_NODE, n, nodes.data()) == SPEX_OK, "fork");
    overwritten = 0;
  }
  spex_status_t append(int n, hipStream_t s) { return spex_tree_append_tokens(t, nodes.data(), n, pool, pool, nullptr, nullptr, s); }
  void end(const char *what) {
    spex_tree_destroy(t);
    run_all();
    CHECK(overwritten == 0, "%s: %ld launches found another list than theirs", what, overwritten);
    queues.clear();
  }
};

int main() {
  hipStream_t one = reinterpret_cast<hipStream_t>(0x100), two = reinterpret_cast<hipStream_t>(0x200);
  queue_behind = {{nullptr, 0}, {one, 1}, {two, 2}};

  // nothing runs until the host waits: many calls ahead, several times round the ring, one stream and two in turn
  for (bool turns : {false, true})
    for (int n : {1, 200, 5000}) {
      Tree t(n);
      waits = 0;
      int ahead = 0;
      for (int i = 0; i < 400; ++i) {
        CHECK(t.append(n, turns && i % 2 ? two : one) == SPEX_OK, "append");
        ahead += waits == 0;
      }
      CHECK(ahead >= 40 && ahead < 400, "%d nodes: %d calls before the host waited", n, ahead);
      t.end(turns ? "two streams" : "one stream");
    }

  // calls that need longer segments while earlier ones wait to run
  {
    Tree t(3000);
    for (int i = 0; i < 60; ++i) CHECK(t.append(10 << (i / 10), i % 3 ? one : two) == SPEX_OK, "append");
    t.end("longer segments");
  }

  // one handle, several streams: each thread's own default stream, and a handle that was destroyed and given out again
  {
    Tree t(200);
    for (int i = 0; i < 400; ++i) {
      thread_now = i % 3;
      CHECK(t.append(200, hipStreamPerThread) == SPEX_OK, "append");
    }
    t.end("streams of threads");
    Tree u(200);
    for (int i = 0; i < 400; ++i) {
      queue_behind[one] = 10 + i / 7;
      CHECK(u.append(200, one) == SPEX_OK, "append");
    }
    u.end("a handle given out again");
  }

  // the event behind a launch cannot be recorded: the call says so, and later ones leave its list alone
  {
    Tree t(200);
    for (int i = 0; i < 400; ++i) {
      records_that_fail = i == 59;
      CHECK(t.append(200, i < 60 ? one : two) == (i == 59 ? SPEX_ERR_DEVICE : SPEX_OK), "call %d", i);
    }
    t.end("an event that was not recorded");
  }

  if (failures == 0) std::printf("ok\n");
  return failures != 0;
}
