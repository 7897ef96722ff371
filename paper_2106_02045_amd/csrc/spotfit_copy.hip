// spotfit_copy.hip -- small copies between pinned host memory and the device as
// a kernel.
//
// A copy of a few KB through the copy engines costs its hand-over: the engine and
// the compute queue wait for each other's signals before and after it.  A kernel
// stays in the queue of the fit it feeds, and copies several arrays in one
// launch.  A captured fit of 32 spots of 13x13, us a replay with the engine / the
// kernel, by the bytes copied in: 16 KB 37.8 / 30.7, 256 KB 41.0 / 34.3, 1 MB
// 58.0 / 47.5, 4 MB 115 / 102.  Larger copies stay with the engine, which leaves
// the compute units to the fits of other streams.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "spotfit_internal.h"

namespace sf {
namespace cpy {

// The host side is read and written past the caches (system scope): a replayed
// launch sees what the host wrote since the last one, whatever kind of pinned
// memory it is, and the host sees the results when the launch is done.
template <typename T>
__device__ __forceinline__ void copy_one(const void* src, void* dst) {
  const T v = __hip_atomic_load(static_cast<const T*>(src), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __hip_atomic_store(static_cast<T*>(dst), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Unit u of the list: 8 bytes of one array, or its last bytes.  One unit per
// thread, so that every load of the launch is in flight at once.
__global__ __launch_bounds__(256) void copy_kernel(CopyList l) {
  int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
  for (int s = 0; s < kCopyMax; ++s) {
    const int64_t units = (l.bytes[s] + 7) >> 3;
    if (u < units) {
      const char* src = static_cast<const char*>(l.src[s]) + 8 * u;
      char* dst = static_cast<char*>(l.dst[s]) + 8 * u;
      const int64_t left = l.bytes[s] - 8 * u;
      const uintptr_t bits = reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst);
      if (left >= 8 && (bits & 7) == 0) {
        copy_one<uint64_t>(src, dst);
      } else {
        const int n = left < 8 ? (int)left : 8;
        int i = 0;
        if ((bits & 3) == 0)
          for (; i + 4 <= n; i += 4) copy_one<uint32_t>(src + i, dst + i);
        for (; i < n; ++i) copy_one<uint8_t>(src + i, dst + i);
      }
      return;
    }
    u -= units;
  }
}

}  // namespace cpy

bool CopyList::add(void* d, const void* s, int64_t n) {
  if (n <= 0) return true;
  if (count == kCopyMax || total + n > kCopyBytes) return false;
  dst[count] = d;
  src[count] = s;
  bytes[count++] = n;
  total += n;
  return true;
}

hipError_t launch_copy(const CopyList& l, hipStream_t st) {
  int64_t units = 0;
  for (int s = 0; s < l.count; ++s) units += (l.bytes[s] + 7) >> 3;
  if (units == 0) return hipSuccess;
  hipLaunchKernelGGL(cpy::copy_kernel, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, st, l);
  return hipGetLastError();
}

// The device's address of n bytes of pinned host memory, or null when they do not
// lie in one pinned allocation.  (Two ends that are pinned say nothing about what
// is between them: a device address is the host's own.)
void* pinned_address(const void* host, int64_t n) {
  hipPointerAttribute_t a;
  hipDeviceptr_t base = nullptr;
  size_t size = 0;
  if (n <= 0 || hipPointerGetAttributes(&a, host) != hipSuccess ||
      hipMemGetAddressRange(&base, &size, const_cast<void*>(host)) != hipSuccess) {
    (void)hipGetLastError();  // an address the runtime does not know
    return nullptr;
  }
  const uintptr_t from = reinterpret_cast<uintptr_t>(host) - reinterpret_cast<uintptr_t>(base);
  if (a.type != hipMemoryTypeHost || !a.devicePointer || from > size || (size_t)n > size - from) return nullptr;
  return a.devicePointer;
}

}  // namespace sf
