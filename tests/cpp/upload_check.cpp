// CPU check of the uploads' route: a kernel that reads the pinned memory
// itself, or the copy engine.  The host code (ss_host.cpp, ss_upload.cpp) is
// linked with stub launchers and a stub HIP runtime that knows a table of
// allocations, records which way each upload goes and can be told to fail.
#include "ss_kernels.h"
#include "specstream.h"

#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

namespace {
int fails = 0;
#define CHECK(c, ...) do { if (!(c)) { printf("FAIL %s:%d: ", __FILE__, __LINE__); printf(__VA_ARGS__); printf("\n"); ++fails; } } while (0)

struct Alloc { uintptr_t at; size_t bytes; hipMemoryType type; int device; unsigned flags; };
constexpr uintptr_t H0 = 0x10000000, H1 = 0x20000000, D0 = 0x200000000000, D1 = 0x210000000000;
constexpr size_t M = 1 << 20;
const Alloc allocs[] = {
    {H0, 8 * M, hipMemoryTypeHost, 0, 0},
    {H0 + 8 * M, 4 * M, hipMemoryTypeHost, 0, 0},              // right behind the first
    {H0 + 16 * M, 4 * M, hipMemoryTypeHost, 0, 0},             // behind a hole
    {H1, 128 * M, hipMemoryTypeHost, 0, 0},
    {H1 + 256 * M, 8 * M, hipMemoryTypeHost, 1, 0},            // pinned for the other GPU
    {H1 + 512 * M, 8 * M, hipMemoryTypeHost, 0, hipHostMallocNonCoherent},
    {H1 + 768 * M, 8 * M, hipMemoryTypeHost, 0, hipHostMallocCoherent},
    {H1 + 1024 * M, 8 * M, hipMemoryTypeHost, 0, hipHostMallocPortable},
    {H1 + 1280 * M, 8 * M, hipMemoryTypeHost, 0, hipHostMallocWriteCombined},
    {H1 + 1536 * M, 8 * M, hipMemoryTypeHost, 0, hipHostMallocMapped | hipHostMallocPortable},
    {H1 + 1792 * M, 8 * M, hipMemoryTypeHost, 0, hipHostMallocMapped | hipHostMallocNonCoherent},
    {D0, 8 * M, hipMemoryTypeDevice, 0, 0},
    {D0 + 8 * M, 8 * M, hipMemoryTypeDevice, 0, 0},
    {D0 + 18 * M, 8 * M, hipMemoryTypeDevice, 0, 0},
    {D1, 128 * M, hipMemoryTypeDevice, 0, 0},
    {D1 + 256 * M, 8 * M, hipMemoryTypeDevice, 1, 0},
};
const Alloc *find(const void *p) {
  for (const Alloc &a : allocs)
    if ((uintptr_t)p >= a.at && (uintptr_t)p < a.at + a.bytes) return &a;
  return nullptr;
}

struct Up { char way; const void *dst, *src; size_t bytes; };   // 'k'ernel or 'e'ngine
std::vector<Up> ups;
int attention = 0, fail_kernel = 0, fail_engine = 0, stream_device = 0;
}  // namespace

namespace ss {
hipError_t launch_chunk(const ChunkParams &, hipStream_t) { ++attention; return hipSuccess; }
hipError_t launch_finalize(const FinalParams &, hipStream_t) { return hipSuccess; }
hipError_t launch_clear_counters(uint32_t *, int, hipStream_t) { return hipSuccess; }
hipError_t launch_read_probe(const void *, uint64_t, uint64_t, uint32_t *, int, hipStream_t) { return hipSuccess; }
hipError_t scratch_address(void **) { return hipErrorNotSupported; }
hipError_t launch_upload(void *dst, const void *src, uint64_t bytes, hipStream_t) {
  ups.push_back({'k', dst, src, bytes});
  return fail_kernel ? hipErrorLaunchFailure : hipSuccess;
}
}  // namespace ss

extern "C" {
const char *hipGetErrorString(hipError_t) { return "stub error"; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned int) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t bytes, hipMemcpyKind, hipStream_t) {
  ups.push_back({'e', dst, src, bytes});
  return fail_engine ? hipErrorInvalidValue : hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  static uintptr_t next = 0x1000;
  *e = reinterpret_cast<hipEvent_t>(next += 0x10);
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t *d) { *d = stream_device; return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
  std::memset(a, 0, sizeof *a);
  const Alloc *f = find(p);
  if (f == nullptr) return hipErrorInvalidValue;
  a->type = f->type;
  a->device = f->device;
  a->devicePointer = const_cast<void *>(p);
  a->allocationFlags = f->flags;
  return hipSuccess;
}
hipError_t hipPointerGetAttribute(void *out, hipPointer_attribute what, hipDeviceptr_t p) {
  const Alloc *f = find(p);
  if (f == nullptr) return hipErrorInvalidValue;
  if (what == HIP_POINTER_ATTRIBUTE_RANGE_START_ADDR) *static_cast<uintptr_t *>(out) = f->at;
  else if (what == HIP_POINTER_ATTRIBUTE_RANGE_SIZE) *static_cast<size_t *>(out) = f->bytes;
  else return hipErrorInvalidValue;
  return hipSuccess;
}
}

namespace {
// the way a pipeline's upload of one chunk of `tokens` tokens (8 KV heads: 4 KiB each) from src to slot dst goes
char way(uintptr_t dst, uintptr_t src, int tokens, ss_status want = SS_OK) {
  const int32_t n_cand = 1, len = tokens;
  ss_round_desc d{};
  d.num_requests = 1; d.num_q_heads = 8; d.num_kv_heads = 8; d.head_dim = 128; d.softmax_scale = 0.1f;
  d.num_cand = &n_cand; d.max_chunk_tokens = 1 << 20;
  ss_round *r = nullptr;
  ss_pipeline *p = nullptr;
  ss_status s = ss_round_init(&r, &d, (void *)0x7f0000000000, (void *)0x7f1000000000, ss_round_workspace_bytes(&d), nullptr);
  if (s == SS_OK) s = ss_pipeline_create(&p, (void *)dst, (void *)(D1 + 64 * M), 1 << 30, nullptr);
  CHECK(s == SS_OK, "set-up: %s", ss_last_error());
  ups.clear();
  attention = 0;
  s = ss_pipeline_attend_chunk(p, r, (const void *)src, &len, nullptr);
  CHECK(s == want, "status %d, want %d: %s", s, want, ss_last_error());
  CHECK(attention == (want == SS_OK), "attention launched %d times", attention);
  CHECK(ups.size() <= 1, "%zu copies", ups.size());
  char w = '-';
  if (!ups.empty()) {
    w = ups[0].way;
    CHECK(ups[0].dst == (void *)dst && ups[0].src == (void *)src && ups[0].bytes == (size_t)tokens * 4096, "copy arguments");
  }
  ss_pipeline_destroy(p);
  ss_round_destroy(r);
  return w;
}
void expect(const char *what, char want, char got) { CHECK(want == got, "%s: went '%c', want '%c'", what, got, want); }
}  // namespace

int main() {
  const int MT = 256;   // tokens a MiB
  expect("inside one allocation", 'k', way(D1, H1, 4 * MT));
  expect("a whole allocation", 'k', way(D0, H0, 8 * MT));
  expect("to the end of one", 'k', way(D0 + 4 * M, H0 + 4 * M, 4 * MT));
  // a range over two allocations, neighbours or with a hole between them, is the copy call's to refuse
  expect("source over two neighbours", 'e', way(D1, H0 + 4 * M, 8 * MT));
  expect("source over a hole", 'e', way(D1, H0 + 10 * M, 8 * MT));
  expect("destination over two neighbours", 'e', way(D0 + 4 * M, H1, 8 * MT));
  expect("destination over a hole", 'e', way(D0 + 12 * M, H1, 8 * MT));
  expect("a source of which only the start is pinned", 'e', way(D1, H0 + 18 * M, 4 * MT));
  fail_engine = 1;
  expect("refused by the copy call", 'e', way(D1, H0 + 10 * M, 8 * MT, SS_ERR_HIP));
  fail_engine = 0;
  // memory that the GPU may cache is the copy engine's: a kernel could read what an earlier one left in the cache
  expect("non-coherent source", 'e', way(D1, H1 + 512 * M, MT));
  expect("explicitly coherent source", 'k', way(D1, H1 + 768 * M, MT));
  // without a word on coherence these follow HIP_HOST_COHERENT
  expect("portable source", 'e', way(D1, H1 + 1024 * M, MT));
  expect("write-combined source", 'e', way(D1, H1 + 1280 * M, MT));
  expect("mapped source", 'k', way(D1, H1 + 1536 * M, MT));
  expect("mapped, non-coherent source", 'e', way(D1, H1 + 1792 * M, MT));
  expect("source 8 bytes off", 'e', way(D1, H1 + 8, MT));
  expect("pinned for another GPU", 'e', way(D1, H1 + 256 * M, MT));
  expect("slot on another GPU", 'e', way(D1 + 256 * M, H1, MT));
  stream_device = 1;
  expect("copy stream of another GPU", 'e', way(D1, H1, MT));
  stream_device = 0;
  // past 16 MiB, and outside the pipeline, uploads keep off the CUs
  expect("16 MiB", 'k', way(D1, H1, 16 * MT));
  expect("16 MiB and a token", 'e', way(D1, H1, 16 * MT + 1));
  for (size_t bytes : {(size_t)16, (size_t)4096, 8 * M}) {
    ups.clear();
    CHECK(ss_upload_chunk((void *)D1, (void *)H1, bytes, nullptr, nullptr, nullptr) == SS_OK, "%s", ss_last_error());
    expect("ss_upload_chunk", 'e', ups.empty() ? '-' : ups[0].way);
  }
  // the upload kernel's launch fails: reported, and nothing attended
  fail_kernel = 1;
  expect("launch failure", 'k', way(D1, H1, MT, SS_ERR_HIP));
  {  // a failed launch behind the slot's free wait leaves the pipeline failed
    const int32_t n_cand = 1, len = MT;
    ss_round_desc d{};
    d.num_requests = 1; d.num_q_heads = 8; d.num_kv_heads = 8; d.head_dim = 128; d.softmax_scale = 0.1f;
    d.num_cand = &n_cand; d.max_chunk_tokens = 1 << 20;
    ss_round *r = nullptr;
    ss_pipeline *p = nullptr;
    CHECK(ss_round_init(&r, &d, (void *)0x7f0000000000, (void *)0x7f1000000000, ss_round_workspace_bytes(&d), nullptr) == SS_OK &&
          ss_pipeline_create(&p, (void *)D1, (void *)(D1 + 64 * M), 8 * M, nullptr) == SS_OK, "set-up");
    CHECK(ss_pipeline_attend_chunk(p, r, (void *)H1, &len, nullptr) == SS_ERR_HIP, "launch failure not reported");
    fail_kernel = 0;   // nothing had been enqueued: both stay usable
    for (int c = 0; c < 2; ++c)
      CHECK(ss_pipeline_attend_chunk(p, r, (void *)H1, &len, nullptr) == SS_OK, "chunk %d: %s", c, ss_last_error());
    fail_kernel = 1;
    CHECK(ss_pipeline_attend_chunk(p, r, (void *)H1, &len, nullptr) == SS_ERR_HIP, "launch failure not reported");
    fail_kernel = 0;
    ups.clear();
    CHECK(ss_pipeline_attend_chunk(p, r, (void *)H1, &len, nullptr) == SS_ERR_BAD_STATE && ups.empty(), "pipeline not failed");
    ss_pipeline_destroy(p);
    ss_round_destroy(r);
  }
  printf("%s\n", fails ? "FAILURES" : "all ok");
  return fails ? 1 : 0;
}
