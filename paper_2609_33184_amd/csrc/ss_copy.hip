// Uploads by kernel: pinned host memory -> device memory, read over the host
// link by the GPU itself.
//
// The link bounds an upload (57.4 GB/s); what it loses is fixed cost.  A copy
// through the copy engine starts about 10 us after its stream is ready, and
// between streams, as in the two-slot pipeline, 20 to 40 us after the event
// it waits for.  A kernel needs neither.  Back to back on one stream, engine
// against kernel: 64 KiB 10.4 -> 4.0 us, 1 MiB 27.3 -> 21.2 us, 8 MiB 156 ->
// 150 us, 32 MiB 596 -> 592 us, 256 MiB 4693 -> 4715 us; a round streamed in
// eight chunks of 8 MiB 1485 -> 1252 us.
#include <hip/hip_runtime.h>

#include "ss_kernels.h"

namespace ss {
namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kCopyThreads = 256;
constexpr int kCopyDepth = 4;      // 16-byte loads in flight per thread
// 16 workgroups keep 256 KiB in flight, which covers the link's latency; more
// only queue up in front of it (the streamed round above: 1252 us with 16, 1280
// with 32, 1283 with 64, 1344 with 128) and take CUs from the attention.
constexpr unsigned kCopyWgs = 16;

__global__ void __launch_bounds__(kCopyThreads) copy_kernel(const u32x4_t *src, u32x4_t *dst, uint64_t n, uint32_t tail) {
  constexpr uint64_t kBlock = (uint64_t)kCopyThreads * kCopyDepth;
  const uint64_t blocks = n / kBlock;
  for (uint64_t b = blockIdx.x; b < blocks; b += gridDim.x) {
    const uint64_t i = b * kBlock + threadIdx.x;
    u32x4_t v[kCopyDepth];
#pragma unroll
    for (int k = 0; k < kCopyDepth; ++k) v[k] = __builtin_nontemporal_load(src + i + k * kCopyThreads);
#pragma unroll
    for (int k = 0; k < kCopyDepth; ++k) dst[i + k * kCopyThreads] = v[k];
  }
  if (blockIdx.x == gridDim.x - 1) {
    for (uint64_t i = blocks * kBlock + threadIdx.x; i < n; i += kCopyThreads) dst[i] = src[i];
    const uint8_t *s8 = reinterpret_cast<const uint8_t *>(src + n);
    uint8_t *d8 = reinterpret_cast<uint8_t *>(dst + n);
    if (threadIdx.x < tail) d8[threadIdx.x] = s8[threadIdx.x];
  }
}

}  // namespace

hipError_t launch_upload(void *dst, const void *mapped_src, uint64_t bytes, hipStream_t s) {
  const uint64_t n = bytes / 16, blocks = n / (kCopyThreads * kCopyDepth);
  const unsigned grid = (unsigned)(blocks < 1 ? 1 : blocks > kCopyWgs ? kCopyWgs : blocks);
  hipLaunchKernelGGL(copy_kernel, dim3(grid), dim3(kCopyThreads), 0, s, static_cast<const u32x4_t *>(mapped_src),
                     static_cast<u32x4_t *>(dst), n, (uint32_t)(bytes % 16));
  return hipGetLastError();
}

}  // namespace ss
