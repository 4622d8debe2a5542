// Which of the pipeline's uploads run as a kernel that reads the pinned memory
// itself (ss_copy.hip); the copy engine takes the others.
//
// The kernel saves the 20 to 40 us after which the engine starts behind another
// stream's event, but it needs CUs: it waits for a workgroup of what fills the
// GPU to end, and slows the rest.  Rounds of 96 MiB streamed in chunks of 4 to
// 32 MiB, engine against kernel in us:
//                       4 MiB        8 MiB       12 MiB       16 MiB       32 MiB
//   alone           2600 2055    2500 1918    2180 1874    1950 1854    1838 1813
//   8192^3 GEMM     3360 2816    3080 2609    2600 2501    2235 2411    1915 2104
//     after each
//   12 layer GEMMs  3160 2639    2820 2470    2700 2420    2275 2389    1930 2266
//     after each
//   that GEMM all   8493 8384    7459 7541
//     the time
//   16 x 32768      2645 2261    2506 2085
//     tokens too
//   the same with   4672 4616    2637 2624
//     64 rows
// so it takes chunks of at most 8 MiB.  Uploads that wait for nothing gain 6 us
// each and lose far more beside other work (8 MiB: 156 and 150 us alone, 156 and
// 596 us beside that GEMM, 157 and 204 us beside 16 x 32768 tokens' attention),
// so ss_upload_chunk leaves them to the engine.
#include "ss_kernels.h"

#include <cstring>

namespace ss {
namespace {

constexpr uint64_t kMaxUpload = uint64_t(8) << 20;

// Non-coherent pinned memory may stay in the GPU's caches from one kernel to the
// next, so that a kernel could read what the host has replaced since.
constexpr unsigned kNonCoherent = hipHostMallocNonCoherent | hipExtHostRegisterCoarseGrained;

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
  if (type == hipMemoryTypeHost && (attr.allocationFlags & kNonCoherent) != 0) return nullptr;
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
