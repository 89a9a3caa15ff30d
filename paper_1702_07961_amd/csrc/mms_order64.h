// Sorting 64-bit keys by 64-bit words that cannot hold them (§6.3 also sorts
// 8-byte integers).
//
// A word is a positive normal double: as integers 2^52 (the smallest) to the
// sentinel, 62 bits for an element's order.  A merge of keys alone whose range is
// below 2^62 has (key - kmin) for its words, kmin and kmax being the tile's
// smallest and largest key.  Otherwise an element's slot in its tile takes 12 of
// the bits, and the words hold the leading 50 of (key - kmin): all of them where
// the range is below 2^50, else keys that agree in those bits (that share a
// prefix) may differ below.  (A base tile first leaves out a run of bits that are
// zero in all of its keys, if the rest then fits.)  The tile is sorted by words,
// and the sorted slots are checked against the keys.  Keys of uniform tiles share
// prefixes about once in 10^8 tiles; a tile that the words did not put in order
// is sorted once more, by words that are exact:
//   bits 37..26  the prefix's rank among the tile's prefixes
//   bits 25..12  the key's bits below the prefix (14 at most)
//   bits 11..0   the slot
// So a tile is sorted at most twice, whatever its keys.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "mms_device.h"
#include "mms_device64.h"
#include "mms_device_kt.h"

namespace mms {

constexpr uint32_t kKeyBits = 62, kSlotBits = 12, kPrefixBits = kKeyBits - kSlotBits;

constexpr uint32_t kWordBase = 1u << 20;   // the smallest normal double's high half

__device__ __forceinline__ uint32_t prefix_shift(uint64_t range) {
    return range >> kPrefixBits ? 64u - kPrefixBits - (uint32_t)__builtin_clzll(range) : 0u;
}
__device__ __forceinline__ double order_word(uint64_t order, uint32_t slot) {
    const uint64_t bits = (order << kSlotBits) | slot;
    return kt_join((uint32_t)(bits >> 32) + kWordBase, (uint32_t)bits);
}
// Words without slots, of which equal ones are equal keys: all 62 bits are the
// key's.
__device__ __forceinline__ double key_word(uint64_t offset) {
    return kt_join((uint32_t)(offset >> 32) + kWordBase, (uint32_t)offset);
}
__device__ __forceinline__ uint64_t word_key(double w) { return (uint64_t)(kt_hi(w) - kWordBase) << 32 | kt_lo(w); }
__device__ __forceinline__ uint32_t word_slot(double w) { return kt_lo(w) & ((1u << kSlotBits) - 1u); }

// op over the 16 lanes of each row (op(x, x) == x).
template <class Op>
__device__ __forceinline__ uint64_t row_reduce(uint64_t x, const Op& op) {
    auto step = [&](auto ctrl) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)x, decltype(ctrl)::value, 0xF, 0xF, false);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(x >> 32), decltype(ctrl)::value, 0xF, 0xF, false);
        const uint64_t o = ((uint64_t)hi << 32) | lo;
        x = op(x, o);
    };
    step(std::integral_constant<int, 0x121>{});   // row_ror:1
    step(std::integral_constant<int, 0x122>{});
    step(std::integral_constant<int, 0x124>{});
    step(std::integral_constant<int, 0x128>{});
    return x;
}
template <bool MAX>
__device__ __forceinline__ uint64_t row_extreme(uint64_t x) {
    return row_reduce(x, [](uint64_t a, uint64_t b) { return MAX ? max(a, b) : min(a, b); });
}
__device__ __forceinline__ uint64_t lane_u64(uint64_t x, int lane) {
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), lane) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, lane);
}

// Keys with a run of bits that are zero in all of them (an id in the high half
// and a counter in the low bits): what is left may fit the 50 bits though the
// range does not.  ones: the OR of the keys; shift: prefix_shift(kmax - kmin), not
// zero.
struct KeyGap {
    uint32_t low, high;   // bits low .. high - 1 are left out
    uint64_t first;       // kmin >> high
    bool fits;
};
__device__ __forceinline__ KeyGap key_gap(uint64_t ones, uint64_t kmin, uint64_t kmax, uint32_t shift) {
    uint64_t runs = ~ones;   // where `have` zeros in a row start
    if ((uint32_t)__popcll(runs) < shift) return {0u, 0u, 0ull, false};   // as of uniform keys, at once
    for (uint32_t have = 1; have < shift;) {
        const uint32_t more = min(have, shift - have);
        runs &= runs >> more;
        have += more;
    }
    const uint32_t low = runs ? (uint32_t)__builtin_ctzll(runs) : 0u;
    const uint64_t above = runs ? ones >> low : 0ull;
    if (!above) return {0u, 0u, 0ull, false};
    const uint32_t high = low + (uint32_t)__builtin_ctzll(above);
    const uint64_t first = kmin >> high, span = (kmax >> high) - first;
    return {low, high, first, low <= kPrefixBits && span >> (kPrefixBits - low) == 0u};
}
__device__ __forceinline__ uint64_t without_gap(uint64_t key, const KeyGap& g) {
    return (((key >> g.high) - g.first) << g.low) | (key & ((1ull << g.low) - 1ull));
}

// LDS of the check and of the second words, for W waves.
template <int W>
struct Order64 {
    uint32_t bad;        // zero before the check
    uint32_t runs[W];    // prefixes that start in each wave's positions

    // Whether the slots in tags (16 bits each, two a word) put the cnt keys of
    // E in the order of (key, slot).  The whole workgroup.
    __device__ __forceinline__ bool ordered(const uint64_t* E, const uint32_t* tags, uint32_t cnt, uint32_t tid) {
        const uint16_t* T = reinterpret_cast<const uint16_t*>(tags);
        auto inverted = [](uint64_t ka, uint32_t a, uint64_t kz, uint32_t z) { return kz < ka || (kz == ka && z < a); };
        bool wrong = false;
        for (uint32_t c = tid; 2u * c + 1u < cnt; c += W * 64u) {
            const uint32_t w = tags[c], a = w & 0xFFFFu, z = w >> 16;
            const uint64_t ka = E[a], kz = E[z];
            wrong = wrong || inverted(ka, a, kz, z);
            if (2u * c + 2u < cnt) {
                const uint32_t y = T[2u * c + 2u];
                wrong = wrong || inverted(kz, z, E[y], y);
            }
        }
        if (__ballot(wrong) && (tid & 63u) == 0u) bad = 1u;
        lds_barrier();
        return __builtin_amdgcn_readfirstlane((int)bad) == 0;
    }

    // Replace every key of E by its second word, in place; every thread takes
    // PER positions in a row (W * 64 * PER >= cnt).  The whole workgroup.
    template <uint32_t PER>
    __device__ __forceinline__ void second_words(uint64_t* E, const uint32_t* tags, uint32_t cnt, uint64_t kmin,
                                                 uint32_t shift, uint32_t tid) {
        // this path is rare: nothing of it is worth a register of the caller's
        // loops, where the compiler would compute it ahead
        asm volatile("" : "+v"(tid));
        const uint16_t* T = reinterpret_cast<const uint16_t*>(tags);
        const uint32_t p0 = tid * PER;
        uint64_t off[PER];
        uint32_t starts = 0;
        uint64_t before = p0 && p0 < cnt ? E[T[p0 - 1u]] - kmin : 0ull;
#pragma unroll
        for (uint32_t j = 0; j < PER; ++j) {
            const uint32_t p = p0 + j;
            off[j] = p < cnt ? E[T[p]] - kmin : 0ull;
            if (p > 0u && p < cnt && (off[j] >> shift) != (before >> shift)) starts |= 1u << j;
            before = off[j];
        }
        // prefixes that start before the thread's positions
        const uint32_t own = (uint32_t)__popc(starts);
        uint32_t run = own;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t o = (uint32_t)__shfl_up((int)run, (unsigned)d, 64);
            if ((int)(tid & 63u) >= d) run += o;
        }
        if ((tid & 63u) == 63u) runs[tid >> 6] = run;
        run -= own;
        lds_barrier();      // every key is read, every wave's count is written
        for (uint32_t w = 0; w < tid >> 6; ++w) run += runs[w];
        double* X = reinterpret_cast<double*>(E);
#pragma unroll
        for (uint32_t j = 0; j < PER; ++j) {
            if (starts & (1u << j)) ++run;
            const uint64_t low = off[j] & ((1ull << shift) - 1ull);
            if (p0 + j < cnt) {
                const uint32_t slot = T[p0 + j];
                X[slot] = order_word(((uint64_t)run << (64u - kPrefixBits)) | low, slot);
            }
        }
    }
};

// Store the cnt keys (or values) of E in the order of tags, each XOR x.  The
// whole workgroup of NT threads.
template <uint32_t NT>
__device__ __forceinline__ void store_by_tags(uint64_t* out, const uint64_t* E, const uint32_t* tags, uint32_t cnt,
                                              uint64_t x, uint32_t tid) {
    typedef uint64_t u64x2 __attribute__((ext_vector_type(2), aligned(8)));
    typedef __attribute__((address_space(1))) u64x2 gu64x2;
    gu64* g = gptr64(out);
    for (uint32_t c = tid; 2u * c < cnt; c += NT) {
        const uint32_t w = tags[c];
        if (2u * c + 1u < cnt) {
            *reinterpret_cast<gu64x2*>(g + 2u * c) = u64x2{E[w & 0xFFFFu] ^ x, E[w >> 16] ^ x};
        } else {
            g[2u * c] = E[w & 0xFFFFu] ^ x;
        }
    }
}

}  // namespace mms
