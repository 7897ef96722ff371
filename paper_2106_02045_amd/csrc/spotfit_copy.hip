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
__device__ __forceinline__ T load_system(const char* p) {
  return __hip_atomic_load(reinterpret_cast<const T*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
template <typename T>
__device__ __forceinline__ void store_system(char* p, T v) {
  __hip_atomic_store(reinterpret_cast<T*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// 8-byte words of the destination that an array touches.
__host__ __device__ __forceinline__ int64_t words_of(const void* dst, int64_t bytes) {
  return bytes > 0 ? (int64_t)(((reinterpret_cast<uintptr_t>(dst) & 7) + (uint64_t)bytes + 7) >> 3) : 0;
}

// One aligned 8-byte word of a destination per thread, so that every access of the
// launch is in flight at once and crosses the bus in whole words.  Where the source
// lies at another place in its words, the thread has the source word that its own
// begins in, and the next one from its neighbour (the last thread of a wavefront or
// array reads it).  What such words would take from outside the array, and the
// ends of one, go byte by byte.  Smaller units for a whole array cost its bus
// accesses many times over: the results of 8,000 spots to host arrays 4 bytes off
// 8-byte alignment took 5046 us a replay by 4-byte units and take 110 (aligned 107,
// the engine 119), of 300 spots 235 and 36.5 (34.4, 48), 512 KB of pixels 2 bytes
// off 109 by bytes and 41 (37.4, 52), 1 KB 39.4 and 32.0 (29.7, 42.7).
__global__ __launch_bounds__(256) void copy_kernel(CopyList l) {
  int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const char* src = nullptr;
  char* dst = nullptr;
  int64_t n = 0;
  int array = 0;  // number of the thread's array, from 1
  for (int s = 0; s < kCopyMax; ++s) {
    const int64_t words = words_of(l.dst[s], l.bytes[s]);
    if (array == 0 && u < words) {
      src = static_cast<const char*>(l.src[s]);
      dst = static_cast<char*>(l.dst[s]);
      n = l.bytes[s];
      array = s + 1;
    }
    if (array == 0) u -= words;
  }
  const int64_t at = 8 * u - (int64_t)(reinterpret_cast<uintptr_t>(dst) & 7);  // the word's place in the array
  const int late = (int)(reinterpret_cast<uintptr_t>(src + at) & 7);  // bytes into a source word
  const bool whole = array != 0 && at >= 0 && at + 8 <= n;
  const bool has = whole && at >= late;  // that source word is inside the array
  uint64_t lo = 0;
  if (has) lo = load_system<uint64_t>(src + (at - late));
  uint64_t hi = __shfl_down(lo, 1);
  const int from = __shfl_down(has ? array : 0, 1);
  bool both = late == 0 || (__lane_id() != 63 && from == array);
  if (has && !both && at - late + 16 <= n) {
    hi = load_system<uint64_t>(src + (at - late) + 8);
    both = true;
  }
  if (has && both) {
    store_system(dst + at, late ? lo >> (8 * late) | hi << (64 - 8 * late) : lo);
  } else if (array != 0) {
    uint8_t b[8];  // all loads at once: a byte outside the array is its nearest one, not stored
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t p = at + i < 0 ? 0 : at + i < n ? at + i : n - 1;
      b[i] = load_system<uint8_t>(src + p);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (at + i >= 0 && at + i < n) store_system(dst + at + i, b[i]);
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
  int64_t words = 0;
  for (int s = 0; s < l.count; ++s) words += cpy::words_of(l.dst[s], l.bytes[s]);
  if (words == 0) return hipSuccess;
  hipLaunchKernelGGL(cpy::copy_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st, l);
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
