// Which uploads run as a kernel that reads the pinned memory itself
// (ss_copy.hip); the copy engine takes the others.
#include "ss_kernels.h"

#include <cstring>

namespace ss {
namespace {

// Larger uploads gain nothing and leave the CUs to others.
constexpr uint64_t kMaxUpload = uint64_t(64) << 20;

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
  if (bytes > kMaxUpload) return nullptr;
  int current = -1;
  hipDevice_t of_stream = -1;
  if (hipGetDevice(&current) != hipSuccess || hipStreamGetDevice(s, &of_stream) != hipSuccess || of_stream != current) {
    (void)hipGetLastError();
    return nullptr;
  }
  return mapped(dst, bytes, hipMemoryTypeDevice, current) == dst ? mapped(src, bytes, hipMemoryTypeHost, current) : nullptr;
}

}  // namespace ss
