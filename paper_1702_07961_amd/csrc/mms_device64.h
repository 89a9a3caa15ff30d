// Element kinds of the 64-bit sorts (§6.3 also sorts 8-byte integers) for
// the generic networks of mms_device.h (the bitonic wave sort and its merge
// across waves).
//
//   E64   a 64-bit key (unsigned order; signed keys are mapped with
//         key ^ 2^63 on the way in and back on the way out)
//   E64T  key and tag.  The tag is the element's slot in the tile as loaded, so
//         (key, tag) is the stable order and every network sorts stably; the
//         values stay in LDS where they were loaded and are gathered by tag
//         when a tile is stored.
//
// Every LDS access of the networks moves one element per lane at
// consecutive element positions (a fixed function of lane and step plus a
// wave-uniform base), so their traffic is free of bank conflicts whatever
// the keys; only the final gather of values by tag reads data-dependent
// addresses.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mms_device.h"

namespace mms {

constexpr uint64_t kSentKey64 = ~0ull;
constexpr uint32_t kSentTag = 0xFFFFFFFFu;   // above every tag

typedef __attribute__((address_space(1))) uint64_t gu64;
typedef const __attribute__((address_space(1))) uint64_t cgu64;
__device__ __forceinline__ gu64* gptr64(uint64_t* p) { return (gu64*)p; }
__device__ __forceinline__ cgu64* gptr64(const uint64_t* p) { return (cgu64*)p; }

struct E64 {
    uint64_t k;
    __device__ static E64 sentinel() { return {kSentKey64}; }
};
struct E64T {
    uint64_t k;
    uint32_t t;
    __device__ static E64T sentinel() { return {kSentKey64, kSentTag}; }
};

__device__ __forceinline__ bool before(const E64T& a, const E64T& b) {
    return a.k < b.k || (a.k == b.k && a.t < b.t);
}

__device__ __forceinline__ void cex(E64& lo, E64& hi) {
    const uint64_t a = lo.k, b = hi.k;
    const bool sw = b < a;
    lo.k = sw ? b : a;
    hi.k = sw ? a : b;
}
__device__ __forceinline__ void cex(E64T& lo, E64T& hi) {
    const bool sw = before(hi, lo);
    const E64T a = lo, b = hi;
    lo.k = sw ? b.k : a.k; lo.t = sw ? b.t : a.t;
    hi.k = sw ? a.k : b.k; hi.t = sw ? a.t : b.t;
}

// keep the earlier (want_first) or the later of `mine` and `other`
__device__ __forceinline__ E64 pick(const E64& mine, const E64& other, bool want_first) {
    const bool other_first = other.k < mine.k;
    return {(want_first ? other_first : !other_first) ? other.k : mine.k};
}
__device__ __forceinline__ E64T pick(const E64T& mine, const E64T& other, bool want_first) {
    const bool other_first = before(other, mine);
    const bool take = want_first ? other_first : !other_first;
    return {take ? other.k : mine.k, take ? other.t : mine.t};
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t x, int m) {
    const uint32_t lo = shfl_xor_u32((uint32_t)x, m);
    const uint32_t hi = shfl_xor_u32((uint32_t)(x >> 32), m);
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ E64 shfl_xor(const E64& e, int m) { return {shfl_xor_u64(e.k, m)}; }
__device__ __forceinline__ E64T shfl_xor(const E64T& e, int m) {
    return {shfl_xor_u64(e.k, m), shfl_xor_u32(e.t, m)};
}

}  // namespace mms
