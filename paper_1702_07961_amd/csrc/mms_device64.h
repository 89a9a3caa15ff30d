// Global-memory views of 64-bit elements (mms_device.h has the 32-bit ones).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mms {

typedef __attribute__((address_space(1))) uint64_t gu64;
typedef const __attribute__((address_space(1))) uint64_t cgu64;
__device__ __forceinline__ gu64* gptr64(uint64_t* p) { return (gu64*)p; }
__device__ __forceinline__ cgu64* gptr64(const uint64_t* p) { return (cgu64*)p; }

}  // namespace mms
