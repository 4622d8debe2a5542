// The two-slot pipeline's small uploads by kernel: pinned host memory -> device
// memory, read over the host link by the GPU itself (ss_upload.cpp has which
// and why).
//
// The link bounds an upload (57.4 GB/s); what it loses is fixed cost.  A copy
// through the copy engine starts 20 to 40 us after the other stream's event it
// waits for, a kernel at once: a round streamed in eight chunks of 8 MiB 1485
// -> 1252 us.
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

__global__ void __launch_bounds__(kCopyThreads) copy_kernel(const u32x4_t *src, u32x4_t *dst, uint64_t n) {
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
  if (blockIdx.x == gridDim.x - 1)
    for (uint64_t i = blocks * kBlock + threadIdx.x; i < n; i += kCopyThreads) dst[i] = src[i];
}

}  // namespace

hipError_t launch_upload(void *dst, const void *mapped_src, uint64_t bytes, hipStream_t s) {
  const uint64_t n = bytes / 16, blocks = n / (kCopyThreads * kCopyDepth);
  const unsigned grid = (unsigned)(blocks < 1 ? 1 : blocks > kCopyWgs ? kCopyWgs : blocks);
  hipLaunchKernelGGL(copy_kernel, dim3(grid), dim3(kCopyThreads), 0, s, static_cast<const u32x4_t *>(mapped_src),
                     static_cast<u32x4_t *>(dst), n);
  return hipGetLastError();
}

}  // namespace ss
