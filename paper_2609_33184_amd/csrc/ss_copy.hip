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

#include <algorithm>

namespace ss {
namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kCopyThreads = 256;
// At most 16 VGPRs a wave (8 of the attribute's units), so that a workgroup
// finds room on a CU that two of the wide history kernel share: two 16-byte
// loads in flight and one offset.  16 workgroups, 128 KiB in flight, cover the
// link's latency on an idle GPU (8 MiB chunks: 1275 us with 16 and with 32, 1291
// with 12, 1490 with 8; more than 256 KiB only queues up in front of the link: 32
// workgroups of four loads 1280, 64 1283, 128 1344 us where 16 took 1252).  32
// hold their own beside other streams' work (a round streamed in 8 MiB chunks
// beside attention 1330 us with 32, 1580 with 16), but what shares a CU with them
// waits longer: many short requests on 1 to 2 MiB of history, whose attention
// takes no longer than the next round's upload, get 16 (51 requests of 1 to 41
// tokens 101 us a round with 32, 84 with 16 and 88 by the copy engine; 32
// requests of 8 tokens 89, 80 and 89; from 4 MiB on 16 and 32 are equal there).
// Between the two, a workgroup per 128 KiB.
constexpr int kCopyDepth = 2;
constexpr unsigned kCopyWgs = 32;
constexpr unsigned kFewCopyWgs = 16;
constexpr unsigned kCopyShare = 128 << 10;
constexpr int kBufferFlags = 0x00020000;   // buffer resource word 3: 32-bit data format, raw offsets
constexpr int kOnce = 2;                   // non-temporal: every byte is read once

__global__ void __launch_bounds__(kCopyThreads) __attribute__((amdgpu_num_vgpr(8))) copy_kernel(const void *src, void *dst,
                                                                                            uint32_t bytes) {
  constexpr uint32_t kRow = kCopyThreads * 16, kBlock = kRow * kCopyDepth;
  const __amdgpu_buffer_rsrc_t from = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(src), (short)0, (int)bytes, kBufferFlags);
  const __amdgpu_buffer_rsrc_t to = __builtin_amdgcn_make_buffer_rsrc(dst, (short)0, (int)bytes, kBufferFlags);
  const uint32_t blocks = bytes / kBlock, t = threadIdx.x * 16;
  for (uint32_t b = blockIdx.x; b < blocks; b += gridDim.x) {
    u32x4_t v[kCopyDepth];
#pragma unroll
    for (int k = 0; k < kCopyDepth; ++k) v[k] = __builtin_amdgcn_raw_buffer_load_b128(from, t, b * kBlock + k * kRow, kOnce);
#pragma unroll
    for (int k = 0; k < kCopyDepth; ++k) __builtin_amdgcn_raw_buffer_store_b128(v[k], to, t, b * kBlock + k * kRow, 0);
  }
  // the rest: words past the end read zero and are not written
  if (blockIdx.x == gridDim.x - 1)
    for (uint32_t o = blocks * kBlock; o < bytes; o += kRow)
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_amdgcn_raw_buffer_load_b128(from, o + t, 0, kOnce), to, o + t, 0, 0);
}

}  // namespace

hipError_t launch_upload(void *dst, const void *mapped_src, uint64_t bytes, hipStream_t s) {
  if (bytes == 0 || bytes % 16 != 0 || bytes >= (uint64_t(1) << 31)) return hipErrorInvalidValue;
  const uint64_t blocks = bytes / (kCopyThreads * 16 * kCopyDepth);
  const uint64_t wgs = std::min<uint64_t>(kCopyWgs, std::max<uint64_t>(kFewCopyWgs, bytes / kCopyShare));
  const unsigned grid = (unsigned)std::max<uint64_t>(1, std::min(wgs, blocks));
  hipLaunchKernelGGL(copy_kernel, dim3(grid), dim3(kCopyThreads), 0, s, mapped_src, dst, (uint32_t)bytes);
  return hipGetLastError();
}

}  // namespace ss
