// 64-bit words of the sorts whose elements are more than a 32-bit key: a
// (key, tag) pair packed into one double.
//
// The merge and base case of the key-value sort order the pairs (key, tag),
// tag being an element's slot in the tile as loaded, which is the stable
// order (§4.2 sorts blocks with bitonic networks, which are not stable on
// keys alone); the values stay in LDS where they were loaded and are
// gathered by tag when a tile is stored.  The pair is packed into the
// mantissa of a positive normal double with a fixed exponent:
//   bits 63..52  0x400 (sign 0, biased exponent 1024)
//   bits 51..20  key
//   bits 19..0   tag (< 2^16 here; the sentinel's is 0xFFFFF)
// Doubles of one sign and exponent order like their mantissas, so the 64-bit
// float min and max (one full-rate instruction each, exact, no rounding) are
// the compare-exchange of the pairs, and the sentinel (key 0xFFFFFFFF, tag
// 0xFFFFF) is above every real element.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mms_device.h"

namespace mms {

constexpr uint32_t kKtExp = 0x400u << 20;   // sign and exponent in the high word

__device__ __forceinline__ double kt_join(uint32_t hi, uint32_t lo) {
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ uint32_t kt_hi(double x) { return (uint32_t)(__builtin_bit_cast(uint64_t, x) >> 32); }
__device__ __forceinline__ uint32_t kt_lo(double x) { return (uint32_t)__builtin_bit_cast(uint64_t, x); }

__device__ __forceinline__ double kt_pack(uint32_t key, uint32_t tag) {
    // high word: exponent | key >> 12; low word: key << 20 | tag
    return kt_join(__builtin_amdgcn_alignbit(0x400u, key, 12u), (key << 20) | tag);
}
__device__ __forceinline__ uint32_t kt_key(double x) { return __builtin_amdgcn_alignbit(kt_hi(x), kt_lo(x), 20u); }
__device__ __forceinline__ uint32_t kt_tag(double x) { return kt_lo(x) & 0xFFFFFu; }
__device__ __forceinline__ double kt_sentinel() { return kt_join(kKtExp | 0xFFFFFu, 0xFFFFFFFFu); }

// min and max as single instructions (the library's fmin would first
// quieten possible signalling NaNs, which these values never are)
__device__ __forceinline__ double kt_min(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double kt_max(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ void cex_kt(double& lo, double& hi) {
    const double a = lo, b = hi;
    lo = kt_min(a, b);
    hi = kt_max(a, b);
}

// A (key, tag) word as an element of the generic networks (wave_sort_blocked,
// wave_merge_tail): compare-exchange by min and max, a lane-dependent pick by
// one compare, and lane exchanges of both halves.
struct ElemKT {
    double d;
    __device__ static ElemKT sentinel() { return {kt_sentinel()}; }
};
__device__ __forceinline__ void cex(ElemKT& lo, ElemKT& hi) { cex_kt(lo.d, hi.d); }
__device__ __forceinline__ ElemKT pick(const ElemKT& mine, const ElemKT& other, bool want_first) {
    const bool other_first = other.d < mine.d;
    return (want_first == other_first) ? other : mine;
}
__device__ __forceinline__ ElemKT shfl_xor(const ElemKT& e, int m) {
    return {kt_join(shfl_xor_u32(kt_hi(e.d), m), shfl_xor_u32(kt_lo(e.d), m))};
}

}  // namespace mms
