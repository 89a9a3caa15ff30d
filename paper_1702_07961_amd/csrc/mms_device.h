// Device building blocks of the multiway mergesort on gfx950 (wave64).
//
// Everything here obeys one rule that makes the LDS traffic free of bank
// conflicts whatever the data: every LDS instruction touches addresses that
// are a fixed function of (lane, step) plus a wave-uniform base.  All
// data-dependent routing happens in registers, through compare-exchange
// networks and cross-lane exchanges (§2.2 and §4.2 of the paper explain why
// data-dependent shared-memory addressing is what costs the pairwise
// mergesorts their bank conflicts).
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
typedef __attribute__((address_space(1))) u32x4 gu32x4;

__device__ __forceinline__ gu32* gptr(uint32_t* p) { return (gu32*)p; }
__device__ __forceinline__ cgu32* gptr(const uint32_t* p) { return (cgu32*)p; }

template <bool P> struct Elem;
template <> struct Elem<false> {
    uint32_t k;
    __device__ static Elem sentinel() { return {kSentKey}; }
};

// strict "a comes before b"
__device__ __forceinline__ bool before(const Elem<false>& a, const Elem<false>& b) { return a.k < b.k; }

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

// ---------------------------------------------------------------------------
// Bitonic merge of 64*EM elements held "striped" (lane l, register e holds
// index e*64 + l): register distances first, then lane distances 32..1.
// ---------------------------------------------------------------------------
template <int EM, class El>
__device__ __forceinline__ void bitonic_merge_striped(El (&m)[EM], int lane) {
#pragma unroll
    for (int d = EM / 2; d >= 1; d >>= 1) {
#pragma unroll
        for (int e = 0; e < EM; ++e)
            if ((e & d) == 0) cex(m[e], m[e | d]);
    }
#pragma unroll
    for (int dl = kWave / 2; dl >= 1; dl >>= 1) {
        const bool lo = (lane & dl) == 0;
#pragma unroll
        for (int e = 0; e < EM; ++e) m[e] = pick(m[e], shfl_xor(m[e], dl), lo);
    }
}

// ---------------------------------------------------------------------------
// Merge-path split inside LDS: the number p of elements of A = X[aA, aA+la)
// among the first d elements of merge(A, B = X[aB, aB+lb)), A first on ties.
// The wave probes 64 points per round, one per lane, with an odd stride, so
// the 64 reads of one round fall in 64 distinct banks (for 64-bit keys, on
// distinct bank pairs: 32 lanes are served per cycle and lane l covers words
// 2(c + l*step) and 2(c + l*step) + 1).  A range of R > 1 candidates takes
// ceil(log64 R) rounds: at most two for every merge tile here.  X is an LDS view
// (key(i)); keys are compared alone, A first on ties, which is the stable
// order of the two runs.
// ---------------------------------------------------------------------------
template <class View>
__device__ __forceinline__ uint32_t lds_corank2_view(const View& X, uint32_t aA, uint32_t la, uint32_t aB,
                                                     uint32_t lb, uint32_t d, int lane) {
    // wave-uniform bounds, kept in scalar registers
    uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(d > lb ? d - lb : 0u));
    uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)min(d, la));
    while (lo < hi) {
        // probe lane sits at lo + lane*step; a probe past hi reads the last
        // valid position instead (every index stays inside both runs) and
        // does not count
        const uint32_t R = hi - lo;
        const uint32_t step = ((R + 63u) >> 6) | 1u;
        const uint32_t m0 = lo + (uint32_t)lane * step;
        const bool v0 = m0 < hi;
        const uint32_t c0 = v0 ? m0 : hi - 1u;
        const bool p0 = v0 && X.key(aA + c0) <= X.key(aB + d - 1u - c0);
        const uint32_t t = (uint32_t)__popcll(__ballot(p0));
        const uint32_t nvalid = (uint32_t)__popcll(__ballot(v0));
        const uint32_t nlo = t > 0 ? lo + (t - 1u) * step + 1u : lo;
        const uint32_t nhi = t < nvalid ? lo + t * step : hi;
        lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)nlo);
        hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)nhi);
    }
    return lo;
}

// lds_corank2_view over a plain array of 32-bit keys.
struct KeysView {
    const uint32_t* k;
    __device__ __forceinline__ uint32_t key(uint32_t i) const { return k[i]; }
};
__device__ __forceinline__ uint32_t lds_corank2(const uint32_t* Xk, uint32_t aA, uint32_t la, uint32_t aB,
                                                uint32_t lb, uint32_t d, int lane) {
    return lds_corank2_view(KeysView{Xk}, aA, la, aB, lb, d, lane);
}

// ---------------------------------------------------------------------------
// Merge outputs [d0, d1) of the pair (A, B) in blocks of N = 64*EM.  Each
// block reads the next N candidates of A (ascending) and of B (descending),
// keeps the smaller of each opposing pair — the N smallest remaining
// elements, as a bitonic sequence — and sorts them with a bitonic merge.
// The number u of A elements kept advances the wave-uniform cursors.  Reads
// are 64 consecutive elements per instruction; writes likewise.
// Positions past the end of A or B read as sentinels; with keys alone a
// sentinel may stand in for an equal real maximum key, which leaves the
// output values unchanged.  X is an LDS view (key / get / put).
// ---------------------------------------------------------------------------
template <int EM, class View, class Sink>
__device__ __forceinline__ void merge_pair_range(const View& X, uint32_t aA, uint32_t la, uint32_t aB, uint32_t lb,
                                                 uint32_t d0, uint32_t d1, const Sink& out, uint32_t out_base,
                                                 int lane) {
    using El = typename View::El;
    constexpr uint32_t N = (uint32_t)kWave * EM;
    if (la == 0 || lb == 0) {   // one run is empty: the other is already in order
        const uint32_t a0 = lb == 0 ? aA : aB;
        for (uint32_t k = d0 + (uint32_t)lane; k < d1; k += (uint32_t)kWave) out.put(out_base + k, X.get(a0 + k));
        return;
    }
    uint32_t p = lds_corank2_view(X, aA, la, aB, lb, d0, lane);
    uint32_t q = d0 - p;
    for (uint32_t o = d0; o < d1; o += N) {
        El m[EM];
        uint32_t u = 0;
#pragma unroll
        for (int e = 0; e < EM; ++e) {
            const uint32_t k = (uint32_t)e * kWave + (uint32_t)lane;
            const uint32_t ia = p + k;
            const uint32_t jb = q + (N - 1u - k);
            const El a = ia < la ? X.get(aA + ia) : El::sentinel();
            const El b = jb < lb ? X.get(aB + jb) : El::sentinel();
            const bool take_a = !before(b, a);
            m[e] = take_a ? a : b;
            u += (uint32_t)__popcll(__ballot(take_a));
        }
        bitonic_merge_striped<EM>(m, lane);
        const uint32_t cnt = min(N, d1 - o);
#pragma unroll
        for (int e = 0; e < EM; ++e) {
            const uint32_t k = (uint32_t)e * kWave + (uint32_t)lane;
            if (k < cnt) out.put(out_base + o + k, m[e]);
        }
        p += u;
        q += N - u;
    }
}

// ---------------------------------------------------------------------------
// One level of the in-LDS merge tree: segments seg(i) = seg0[min(i<<lvl,
// nseg0)] are merged in adjacent pairs; wave w produces the outputs
// [w*total/nw, (w+1)*total/nw) of the whole level, so the work is balanced
// whatever the segment lengths.
// ---------------------------------------------------------------------------
template <int EM, class View, class Sink>
__device__ __forceinline__ void merge_level(const View& X, const uint32_t* seg0, uint32_t nseg0, uint32_t lvl,
                                            uint32_t total, const Sink& out, int wave, int nwaves, int lane) {
    // total < 2^20 here, so the 32-bit products cannot overflow
    const uint32_t o0 = total * (uint32_t)wave / (uint32_t)nwaves;
    const uint32_t o1 = total * (uint32_t)(wave + 1) / (uint32_t)nwaves;
    const uint32_t nseg = (nseg0 + (1u << lvl) - 1u) >> lvl;
    const uint32_t npairs = (nseg + 1u) / 2u;
    for (uint32_t i = 0; i < npairs; ++i) {
        const uint32_t s0 = seg0[min((2u * i) << lvl, nseg0)];
        const uint32_t s1 = seg0[min((2u * i + 1u) << lvl, nseg0)];
        const uint32_t s2 = seg0[min((2u * i + 2u) << lvl, nseg0)];
        const uint32_t lo = max(o0, s0), hi = min(o1, s2);
        if (lo >= hi) continue;
        merge_pair_range<EM>(X, s0, s1 - s0, s1, s2 - s1, lo - s0, hi - s0, out, s0, lane);
    }
}

// ===========================================================================
// Block merge with LDS transposes (64-bit words: mms_device_kt.h).
//
// The bitonic block of N = 64*EM words is sorted with every compare-exchange
// inside a lane.  Index bits are moved between register and lane positions
// by two transposes through a wave-private scratch whose 64-word rows are
// padded (row stride RS), which makes every scratch access conflict-free:
//   S  (as read)   register = index bits above 6, lane = bits 5..0
//   T1             register = bits 5..3
//   F  (as stored) register 4c+j = position c*256 + 4*lane + j, so each
//                  lane stores 16-byte chunks and a wave stores 1 KiB runs
// Index bit 2 is lane bit 0 in F and takes one DPP exchange.
// Measured gfx950 rules behind the padding: 32-bit accesses are served 32
// lanes per cycle over 32 banks, 128-bit accesses 16 lanes per cycle over 64
// banks.
// ===========================================================================
template <int EM> struct Xpose;
template <> struct Xpose<8> {
    static constexpr uint32_t RS = 72;
    static constexpr uint32_t WORDS = 8 * RS;
};

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

// Store a block held in layout F: chunk c of lane l is block positions
// p = c*256 + 4l .. p+3.  put4(c, p) stores a whole chunk, put1(c, j, p + j)
// one position; positions at or past lim are not stored, and whole chunks
// only where vec allows it.  A whole block takes one wave-uniform branch.
template <int EM, class Put4, class Put1>
__device__ __forceinline__ void store_block(uint32_t lim, bool vec, int lane, const Put4& put4, const Put1& put1) {
    if (vec && lim >= (uint32_t)EM * 64u) {
#pragma unroll
        for (int c = 0; c < EM / 4; ++c) put4(c, (uint32_t)c * 256u + 4u * (uint32_t)lane);
        return;
    }
#pragma unroll
    for (int c = 0; c < EM / 4; ++c) {
        const uint32_t p = (uint32_t)c * 256u + 4u * (uint32_t)lane;
        if (vec && p + 4u <= lim) {
            put4(c, p);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (p + (uint32_t)j < lim) put1(c, j, p + (uint32_t)j);
        }
    }
}

}  // namespace mms
