// Device building blocks of the multiway mergesort on gfx950 (wave64).
//
// Exchanges and changes of layout touch LDS at addresses that are a fixed
// function of (lane, step) plus a wave-uniform base, and elements are ordered in
// registers, by compare-exchange networks and cross-lane exchanges (§2.2 and
// §4.2 of the paper explain why data-dependent shared-memory addressing is what
// costs the pairwise mergesorts their bank conflicts).  What does depend on the
// data is where a merge block's rows start in their runs and the gather of
// values by tag; these conflict, at 9 to 39 % of a kernel's LDS cycles.
//
// Element kinds: Elem<false> is a 32-bit key (unsigned order; signed keys
// are mapped with key ^ 0x80000000 on the way in and back on the way out).
// Key-value sorts use the (key, tag) words of mms_device_kt.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mms {

constexpr int kWave = 64;
constexpr uint32_t kSentKey = 0xFFFFFFFFu;

// Global-memory views.  Accesses through generic pointers compile to FLAT
// instructions, which count against the LDS counter as well as the vector
// memory counter, so an LDS barrier would wait for them; through
// address-space-1 pointers they become global_* instructions.
typedef __attribute__((address_space(1))) uint32_t gu32;
typedef const __attribute__((address_space(1))) uint32_t cgu32;
// four keys at a 4-byte aligned global address
typedef uint32_t u32x4a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef const __attribute__((address_space(1))) u32x4a4 cgu32x4a4;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// four or two keys stored at a 4-byte aligned address (a batch's segments start
// anywhere): one instruction, like the loads above
typedef __attribute__((address_space(1))) u32x4a4 gu32x4a4;
typedef uint32_t u32x2a4 __attribute__((ext_vector_type(2), aligned(4)));
typedef __attribute__((address_space(1))) u32x2a4 gu32x2a4;

__device__ __forceinline__ gu32* gptr(uint32_t* p) { return (gu32*)p; }
__device__ __forceinline__ cgu32* gptr(const uint32_t* p) { return (cgu32*)p; }

template <bool P> struct Elem;
template <> struct Elem<false> {
    uint32_t k;
    __device__ static Elem sentinel() { return {kSentKey}; }
};

// compare-exchange: lo receives the earlier element, hi the later one
__device__ __forceinline__ void cex(Elem<false>& lo, Elem<false>& hi) {
    uint32_t a = lo.k, b = hi.k;
    lo.k = min(a, b);
    hi.k = max(a, b);
}

// Median of three unsigned values in one instruction: with c = 0 it is
// min(a, b), with c = ~0 it is max(a, b), so a lane-dependent c picks the
// lower or upper half of a compare-exchange without a select.
__device__ __forceinline__ uint32_t med3_u32(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t d;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

__device__ __forceinline__ uint32_t min3_u32(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t d;
    asm("v_min3_u32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
__device__ __forceinline__ uint32_t max3_u32(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t d;
    asm("v_max3_u32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// Two stages of a bitonic merge on four elements of a bitonic sequence at
// equal distances, in six instructions instead of eight.  With lo / hi the
// smaller and larger of a and c, the first stage leaves {lo, min(b, d)} below
// {hi, max(b, d)} element by element, so lo <= max(b, d) and hi >= min(b, d):
// the four results are the minimum and median of (lo, b, d) and the median
// and maximum of (hi, b, d).
__device__ __forceinline__ void bitonic4(uint32_t& a, uint32_t& b, uint32_t& c, uint32_t& d) {
    const uint32_t lo = min(a, c), hi = max(a, c), x = b, y = d;
    a = min3_u32(lo, x, y);
    b = med3_u32(lo, x, y);
    c = med3_u32(hi, x, y);
    d = max3_u32(hi, x, y);
}

// keep the earlier (want_first) or the later of `mine` and `other`
__device__ __forceinline__ Elem<false> pick(const Elem<false>& mine, const Elem<false>& other, bool want_first) {
    return {med3_u32(mine.k, other.k, want_first ? 0u : ~0u)};
}

// Value of lane (lane ^ m).  When m is a constant (after loop unrolling)
// this folds to one exchange: DPP within a row of 16 lanes
// (quad permutes, row mirrors, rotate by 8), a ds_swizzle inside 32 lanes,
// and ds_bpermute across the halves of the wave.
__device__ __forceinline__ uint32_t shfl_xor_u32(uint32_t x, int m) {
    const int v = (int)x;
    // a mask only known at run time (a loop the compiler kept rolled) takes
    // the general permute rather than a branch per exchange
    if (!__builtin_constant_p(m)) return (uint32_t)__shfl_xor(v, m, kWave);
    switch (m) {
        case 1: return (uint32_t)__builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, false);    // quad_perm [1,0,3,2]
        case 2: return (uint32_t)__builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, false);    // quad_perm [2,3,0,1]
        case 3: return (uint32_t)__builtin_amdgcn_mov_dpp(v, 0x1B, 0xF, 0xF, false);    // quad_perm [3,2,1,0]
        case 7: return (uint32_t)__builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, false);   // row_half_mirror
        case 8: return (uint32_t)__builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, false);   // row_ror:8
        case 15: return (uint32_t)__builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, false);  // row_mirror
        // bit-mask swizzle inside 32 lanes: and 0x1F, or 0, xor m
        case 4: return (uint32_t)__builtin_amdgcn_ds_swizzle(v, 0x1F | (4 << 10));
        case 16: return (uint32_t)__builtin_amdgcn_ds_swizzle(v, 0x1F | (16 << 10));
        case 31: return (uint32_t)__builtin_amdgcn_ds_swizzle(v, 0x1F | (31 << 10));
        default: return (uint32_t)__shfl_xor(v, m, kWave);
    }
}
__device__ __forceinline__ Elem<false> shfl_xor(const Elem<false>& e, int m) { return {shfl_xor_u32(e.k, m)}; }

// ---------------------------------------------------------------------------
// Base case: sort the 64*E elements a wave holds, E per lane (§4.3 sorts a
// W x W grid with rows in registers and transposes; here every stage is a
// bitonic compare-exchange, in-lane for index bits below log2(E) and across
// lanes for the rest).  Result layout is "blocked": lane l holds positions
// l*E .. l*E+E-1 of the wave's sorted run.
// ---------------------------------------------------------------------------
template <int E, class El>
__device__ __forceinline__ void wave_sort_blocked(El (&r)[E], int lane) {
#pragma unroll
    for (int s = 1; s < E; s <<= 1) {
#pragma unroll
        for (int e = 0; e < E; ++e)
            if ((e & s) == 0) cex(r[e], r[e ^ (2 * s - 1)]);
#pragma unroll
        for (int d = s / 2; d >= 1; d >>= 1) {
#pragma unroll
            for (int e = 0; e < E; ++e)
                if ((e & d) == 0) cex(r[e], r[e | d]);
        }
    }
#pragma unroll
    for (int sl = 1; sl < kWave; sl <<= 1) {
        // mirror stage: (lane, e) meets (lane ^ (2sl-1), E-1-e)
        const bool lower = (lane & sl) == 0;
        El t[E];
#pragma unroll
        for (int e = 0; e < E; ++e) t[e] = pick(r[e], shfl_xor(r[E - 1 - e], 2 * sl - 1), lower);
#pragma unroll
        for (int e = 0; e < E; ++e) r[e] = t[e];
#pragma unroll
        for (int dl = sl / 2; dl >= 1; dl >>= 1) {
            const bool lo = (lane & dl) == 0;
#pragma unroll
            for (int e = 0; e < E; ++e) r[e] = pick(r[e], shfl_xor(r[e], dl), lo);
        }
#pragma unroll
        for (int d = E / 2; d >= 1; d >>= 1) {
#pragma unroll
            for (int e = 0; e < E; ++e)
                if ((e & d) == 0) cex(r[e], r[e | d]);
        }
    }
}

// The in-wave tail of a bitonic merge in the blocked layout: lane distances
// 32 .. 1, then register distances (after the cross-wave stages of a
// workgroup-wide merge).
template <int E, class El>
__device__ __forceinline__ void wave_merge_tail(El (&r)[E], int lane) {
#pragma unroll
    for (int dl = kWave / 2; dl >= 1; dl >>= 1) {
        const bool lo = (lane & dl) == 0;
#pragma unroll
        for (int e = 0; e < E; ++e) r[e] = pick(r[e], shfl_xor(r[e], dl), lo);
    }
#pragma unroll
    for (int d = E / 2; d >= 1; d >>= 1) {
#pragma unroll
        for (int e = 0; e < E; ++e)
            if ((e & d) == 0) cex(r[e], r[e | d]);
    }
}

// floor(a / b) for b > 0, a < 2^24 and a / b < 2^22, without the integer
// division sequence.  a converts to float exactly; the reciprocal is within
// one ulp and the product rounds once, so the estimate is within
// (a / b) * 2^-22 < 1 of a / b and its truncation within one of the
// quotient; one correction step each way makes it exact (q * b <= a + b
// stays below 2^32).
__device__ __forceinline__ uint32_t udiv_small(uint32_t a, uint32_t b) {
    uint32_t q = (uint32_t)((float)a * __builtin_amdgcn_rcpf((float)b));
    if (q * b > a) --q;
    else if ((q + 1u) * b <= a) ++q;
    return q;
}

// Ordering point for a wave's own LDS traffic.  The LDS performs a wave's
// operations in the order the wave issues them, so a read issued after the
// wave's own writes returns what they wrote without waiting for them to
// complete (the compiler's memory model emits no wait for a fence at
// wavefront scope either); only the compiler must keep the order.
__device__ __forceinline__ void lds_wave_sync() { asm volatile("" ::: "memory"); }

// Wait until every vector memory operation the wave has issued (loads,
// stores, copies into LDS) is complete.
__device__ __forceinline__ void vm_drain() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Copy word `off` of the wave-uniform global array `base` into word `off` of
// the wave-uniform LDS array `lds` through the memory unit (no register
// holds it): one call per lane, lane l passing off = l, moves 64 consecutive
// words.  The copy is complete once the wave's vector memory counter drains.
__device__ __forceinline__ void dma_dword(const uint32_t* base, uint32_t off, uint32_t* lds) {
    const uint64_t a = (uint64_t)(uintptr_t)base;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
    const uint32_t* ub = (const uint32_t*)(uintptr_t)(((uint64_t)hi << 32) | lo);
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(ub + off),
                                     (__attribute__((address_space(3))) void*)lds, 4, 0, 0);
}

// Workgroup barrier for LDS traffic only.  Unlike __syncthreads() it does not
// wait for outstanding global loads and stores, so a prefetch into registers
// and the previous tile's stores stay in flight across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ void cex_u32(uint32_t& lo, uint32_t& hi) {
    const uint32_t a = lo, b = hi;
    lo = min(a, b);
    hi = max(a, b);
}

}  // namespace mms
