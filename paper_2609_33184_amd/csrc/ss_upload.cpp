// Which of the pipeline's uploads run as a kernel that reads the pinned memory
// itself (ss_copy.hip); the copy engine takes the others.
//
// The kernel saves what the engine loses behind another stream's event, 20 us
// and more a chunk.  But it needs CUs, it waits for a workgroup of what fills
// the GPU to end, and what shares a CU with it waits behind its reads over the
// link (a 48 us GEMM ends with the upload beside it).  Rounds of 80 to 96 MiB,
// one request streamed in chunks of the sizes below, engine and kernel in us:
//                          8 MiB      16 MiB     20 MiB     24 MiB     32 MiB
//   alone                2810 1915  2250 1918  1620 1526  1870 1825  1838 1810
//   a GEMM after each    2940 2590  3000 2735  1715 1990  1966 2220  1889 2064
//   12 layer GEMMs each  2730 2460  3100 2518  1910 2018  2150 2300  1961 2242
//   beside that GEMM     7459 7541
//   beside attention     2506 2085
//     of 64 rows         2637 2624
// (GEMMs 8192^3 and 256 x 4096 x 14336; attention of 16 x 32768 tokens), so it
// takes chunks of at most 16 MiB.  A copy stream that shares one of the four
// hardware queues with a stream full of attention launches is the exception:
// engine and kernel 2490 and 2983 us there (8 MiB chunks, the attention of 4 x
// 32768 tokens), 1605 and 1326 on a queue of its own, 1776 and 1529 on that of
// the round's stream; with 2 MiB chunks 990 and 1272, 540 and 533, 744 and 737.
// Uploads that wait for nothing gain 6 us each
// and lose far more beside other work (8 MiB: 156 and 150 us alone, 156 and 596
// us beside the GEMM, 157 and 204 us beside the attention), so ss_upload_chunk
// leaves them to the engine.
#include "ss_kernels.h"

#include <cstring>

namespace ss {
namespace {

constexpr uint64_t kMaxUpload = uint64_t(16) << 20;

// Non-coherent pinned memory may stay in the GPU's caches from one kernel to the
// next, so that a kernel could read what the host has replaced since.  Default
// memory (no flag; torch's pinned tensors) is coherent, and so is what these
// flags ask for; with others (portable, write-combined, NUMA policy) that is
// HIP_HOST_COHERENT's matter, which the allocation's flags don't show.
constexpr unsigned kCoherent = hipHostMallocCoherent | hipHostMallocMapped | hipHostMallocUncached;
constexpr unsigned kNonCoherent = hipHostMallocNonCoherent | hipExtHostRegisterCoarseGrained;
bool coherent(unsigned flags) { return flags == 0 || ((flags & kCoherent) != 0 && (flags & kNonCoherent) == 0); }

// The address at which GPU `device` sees [p, p + bytes), if the range lies
// inside one allocation of the wanted type there and is 16-byte aligned; else
// null.  Neighbouring addresses prove nothing: a range over two allocations
// may have a hole between them, or end in another buffer, and only the copy
// call can refuse it.
const void *mapped(const void *p, uint64_t bytes, hipMemoryType type, int device) {
  hipPointerAttribute_t attr;
  std::memset(&attr, 0, sizeof attr);
  void *start = nullptr;
  size_t size = 0;
  hipDeviceptr_t q = const_cast<void *>(p);
  if (hipPointerGetAttributes(&attr, p) != hipSuccess ||
      hipPointerGetAttribute(&start, HIP_POINTER_ATTRIBUTE_RANGE_START_ADDR, q) != hipSuccess ||
      hipPointerGetAttribute(&size, HIP_POINTER_ATTRIBUTE_RANGE_SIZE, q) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  const uintptr_t d = reinterpret_cast<uintptr_t>(attr.devicePointer), s = reinterpret_cast<uintptr_t>(start);
  if (type == hipMemoryTypeHost && !coherent(attr.allocationFlags)) return nullptr;
  const bool whole = d != 0 && d >= s && d - s <= size && bytes <= size - (d - s);
  return whole && attr.type == type && attr.device == device && d % 16 == 0 ? attr.devicePointer : nullptr;
}

}  // namespace

const void *upload_source(const void *dst, const void *src, uint64_t bytes, hipStream_t s) {
  if (bytes > kMaxUpload || bytes % 16 != 0) return nullptr;
  int current = -1;
  hipDevice_t of_stream = -1;
  if (hipGetDevice(&current) != hipSuccess || hipStreamGetDevice(s, &of_stream) != hipSuccess || of_stream != current) {
    (void)hipGetLastError();
    return nullptr;
  }
  return mapped(dst, bytes, hipMemoryTypeDevice, current) == dst ? mapped(src, bytes, hipMemoryTypeHost, current) : nullptr;
}

}  // namespace ss
