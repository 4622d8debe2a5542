// CPU check of what a thread keeps between calls: the planner's tables stay
// for ordinary calls and are given back after unusually large ones, whether
// the call succeeds, is refused or runs out of memory.
#include "ss_kernels.h"
#include "specstream.h"

#include <malloc.h>

#include <cstdio>
#include <cstdlib>
#include <new>
#include <thread>
#include <vector>

namespace {
long g_live = 0, g_news = 0, g_fail_at = -1;   // heap bytes in use, allocations so far, allocation to fail
int fails = 0;
#define CHECK(c, ...) do { if (!(c)) { printf("FAIL %s:%d: ", __FILE__, __LINE__); printf(__VA_ARGS__); printf("\n"); ++fails; } } while (0)
}  // namespace

void *operator new(size_t n) {
  if (g_news++ == g_fail_at) throw std::bad_alloc();
  void *p = std::malloc(n ? n : 1);
  if (p == nullptr) throw std::bad_alloc();
  g_live += (long)malloc_usable_size(p);
  return p;
}
void operator delete(void *p) noexcept {
  if (p != nullptr) g_live -= (long)malloc_usable_size(p);
  std::free(p);
}
void operator delete(void *p, size_t) noexcept { operator delete(p); }

namespace ss {
hipError_t launch_chunk(const ChunkParams &, hipStream_t) { return hipSuccess; }
hipError_t launch_finalize(const FinalParams &, hipStream_t) { return hipSuccess; }
hipError_t launch_clear_counters(uint32_t *, int, hipStream_t) { return hipSuccess; }
hipError_t launch_read_probe(const void *, uint64_t, uint64_t, uint32_t *, int, hipStream_t) { return hipSuccess; }
hipError_t scratch_address(void **) { return hipErrorNotSupported; }
}  // namespace ss

namespace {
// a round of B requests x 64 tokens in nch chunks of one call
ss_status call(int B, int nch) {
  std::vector<int32_t> cand(B, 1), len((size_t)B * nch, 64 / nch);
  std::vector<const void *> k(nch, (const void *)0x100000000), v(nch, (const void *)0x200000000);
  ss_round_desc d{};
  d.num_requests = B; d.num_q_heads = 2; d.num_kv_heads = 1; d.head_dim = 128; d.softmax_scale = 0.1f;
  d.num_cand = cand.data(); d.max_chunk_tokens = 1 << 30;
  ss_round *r = nullptr;
  ss_status s = ss_round_init(&r, &d, (void *)0x7f0000000000, (void *)0x7f1000000000, ss_round_workspace_bytes(&d), nullptr);
  if (s == SS_OK) s = ss_attend_history_chunks(r, nch, k.data(), v.data(), len.data(), nullptr, nullptr, nullptr);
  ss_round_destroy(r);
  return s;
}
}  // namespace

int main() {
  constexpr long kKeep = 1 << 20;
  std::thread([&] {
    const long before = g_live;
    CHECK(call(64, 16) == SS_OK, "%s", ss_last_error());
    const long small = g_live - before;
    CHECK(small > 0 && small <= kKeep, "an ordinary call keeps %ld bytes", small);
    const long news = g_news;
    CHECK(call(64, 16) == SS_OK, "%s", ss_last_error());
    // the call's own vectors above and the round, but no table of the planner
    CHECK(g_news - news <= 10, "a repeated call makes %ld allocations", g_news - news);
    CHECK(call(40000, 8) == SS_OK, "%s", ss_last_error());
    CHECK(g_live - before <= kKeep, "a large call leaves %ld bytes", g_live - before);
    for (long at = 0; at < 60; at += 3) {
      g_news = 0;
      g_fail_at = 12 + at;
      try {
        (void)call(40000, 8);
      } catch (const std::bad_alloc &) {   // of the vectors above
      }
      g_fail_at = -1;
      CHECK(g_live - before <= kKeep, "out of memory at allocation %ld: %ld bytes left", 12 + at, g_live - before);
    }
    CHECK(call(64, 16) == SS_OK, "%s", ss_last_error());
  }).join();
  printf("%s\n", fails ? "FAILURES" : "all ok");
  return fails ? 1 : 0;
}
