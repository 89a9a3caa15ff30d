// Bitonic sort of a base-case tile (§4.3) with every compare-exchange of
// distance 16 or more moved into registers.
//
// A tile of 1024*W words is sorted by W waves of 16 words per lane.  Word i of
// the tile is named by its index bits; a layout says which of them are
// register bits (four), which lane bits (six) and which wave bits, and moves
// between layouts go through LDS.  A merge step of 2^s words takes its index
// bits s-1 .. 0 four at a time, each four as register bits:
//   s <= 4      in registers (layout A)
//   s = 5, 6    index bits 4 and 5 are lane bits 0 and 1 of A: quad_perm
//   s = 7 .. 10 A -> B(s) (register bits s-1 .. s-4) -> A, inside the wave;
//               bits 5 and 4 by quad_perm where they are left over
//   s > 10      A -> C(s) (register bits s-1 .. s-4) -> D(s) (the next four)
//               -> A; C and D have w = s - 10 low index bits as wave bits
// An exchange across lanes costs two to three VALU instructions a word more
// than one in a register (two moves and a select for 64-bit words), and an
// exchange of every word with a partner wave's through LDS moves it as far as
// a change of layout, which then serves four index bits.
//
// In LDS a 32-bit word i sits at i + (i >> 5) + (i >> 10): index bit i has the
// bank weight 2^(i mod 5), and lane bits 0..4 of every layout are index bits of
// different weights, so all accesses are free of bank conflicts (the counter reads
// zero).  For 64-bit words the writes decide (16 lanes at a time over 32 banks; 6.1
// cycles for 64 lanes against 8.2 with two lanes on a bank, while 64-bit reads take
// 2.5 either way; the counter reads 1.1 cycles an LDS instruction of the pairs' base
// case, its gather by tag among them, and 1.9 with stride-64 keys),
// and i + (i >> 4) + (i >> 8) + (i >> 12) gives weights 2^(i mod 4), and lane
// bits 0..3 are index bits of different ones.  A word's address is the sum of
// its lane's and its register's, the latter a constant.
//
// The first stage of a step pairs i with its mirror in the other half: where
// the top bit is a register bit, those registers read the mirrored place.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mms_device.h"
#include "mms_device_kt.h"

namespace mms {

constexpr int kNetRegs = 16;
template <class T>
constexpr uint32_t net_addr(uint32_t i) {
    return sizeof(T) == 4 ? i + (i >> 5) + (i >> 10) : i + (i >> 4) + (i >> 8) + (i >> 12);
}
// LDS words of a tile
template <class T>
constexpr uint32_t net_words(uint32_t n) {
    return net_addr<T>(n - 1u) + 1u;
}

// ---- words ----------------------------------------------------------------------
struct NetKey {   // 32-bit keys
    using T = uint32_t;
    static __device__ __forceinline__ T sentinel() { return kSentKey; }
    static __device__ __forceinline__ void cex(T& a, T& b) { cex_u32(a, b); }
    static __device__ __forceinline__ void cex4(T& a, T& b, T& c, T& d) { bitonic4(a, b, c, d); }
    template <int CTRL>
    static __device__ __forceinline__ T dpp(T x) {
        return (T)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xF, 0xF, false);
    }
    static __device__ __forceinline__ void keep(T (&m)[kNetRegs], const T (&o)[kNetRegs], bool upper) {
        const uint32_t k = upper ? ~0u : 0u;
#pragma unroll
        for (int e = 0; e < kNetRegs; ++e) m[e] = med3_u32(m[e], o[e], k);
    }
};
struct NetWord {   // 64-bit words (mms_device_kt.h)
    using T = double;
    static __device__ __forceinline__ T sentinel() { return kt_sentinel(); }
    static __device__ __forceinline__ void cex(T& a, T& b) { cex_kt(a, b); }
    static __device__ __forceinline__ void cex4(T& a, T& b, T& c, T& d) {
        cex_kt(a, c);
        cex_kt(b, d);
        cex_kt(a, b);
        cex_kt(c, d);
    }
    template <int CTRL>
    static __device__ __forceinline__ T dpp(T x) {
        return kt_join((uint32_t)__builtin_amdgcn_mov_dpp((int)kt_hi(x), CTRL, 0xF, 0xF, false),
                       (uint32_t)__builtin_amdgcn_mov_dpp((int)kt_lo(x), CTRL, 0xF, 0xF, false));
    }
    static __device__ __forceinline__ void keep(T (&m)[kNetRegs], const T (&o)[kNetRegs], bool upper) {
        if (upper) {
#pragma unroll
            for (int e = 0; e < kNetRegs; ++e) m[e] = kt_max(m[e], o[e]);
        } else {
#pragma unroll
            for (int e = 0; e < kNetRegs; ++e) m[e] = kt_min(m[e], o[e]);
        }
    }
};

// ---- layouts --------------------------------------------------------------------
// kLow: the lowest register bit, the others follow it; lane: the index bits of a
// lane and wave (32-bit words: B's index bit of the weight that lane bits 0..4
// have already is lane bit 5).
template <class T>
struct NetA {
    static constexpr uint32_t kLow = 0;
    static __device__ __forceinline__ uint32_t lane(uint32_t l, uint32_t w) { return (l << 4) | (w << 10); }
};
template <class T, int S>
struct NetB {
    static constexpr uint32_t kLow = S - 4;
    static __device__ __forceinline__ uint32_t lane(uint32_t l, uint32_t w) {
        constexpr uint32_t a = kLow;
        uint32_t i;
        if constexpr (a == 6) i = l;
        else if constexpr (sizeof(T) == 8) i = (l & ((1u << a) - 1u)) | ((l >> a) << (a + 4u));
        else i = (l & ((1u << a) - 1u)) | (((l >> a) & ((1u << (5u - a)) - 1u)) << (a + 5u)) | ((l >> 5) << (a + 4u));
        return i | (w << 10);
    }
};
template <class T, int S>
struct NetC {
    static constexpr uint32_t kLow = S - 4;
    static __device__ __forceinline__ uint32_t lane(uint32_t l, uint32_t w) {
        constexpr uint32_t b = S - 10;
        return (l << b) | (w & ((1u << b) - 1u)) | ((w >> b) << S);
    }
};
template <class T, int S>
struct NetD {
    static constexpr uint32_t kLow = S - 8;
    static __device__ __forceinline__ uint32_t lane(uint32_t l, uint32_t w) {
        constexpr uint32_t b = S - 10;
        const uint32_t hi = sizeof(T) == 8 ? (l >> 2) << (b + 6u) : (((l >> 2) & 7u) << (b + 7u)) | ((l >> 5) << (b + 6u));
        return ((l & 3u) << b) | hi | (w & ((1u << b) - 1u)) | ((w >> b) << S);
    }
};

// 64-bit accesses are kept apart: two in one instruction (ds_read2_b64) take
// 8.5 cycles or more where two single reads take five.
template <class T>
__device__ __forceinline__ void net_single() {
    if (sizeof(T) == 8) asm volatile("" ::: "memory");
}

template <class Lay, class T>
__device__ __forceinline__ void net_put(T* X, const T (&m)[kNetRegs], uint32_t l, uint32_t w) {
    T* p = X + net_addr<T>(Lay::lane(l, w));
#pragma unroll
    for (uint32_t r = 0; r < kNetRegs; ++r) {
        p[net_addr<T>(r << Lay::kLow)] = m[r];
        net_single<T>();
    }
}
// S > 0: registers with index bit S-1 read the mirrored place (bits S-2 .. 0
// inverted).
template <class Lay, int S, class T>
__device__ __forceinline__ void net_get(const T* X, T (&m)[kNetRegs], uint32_t l, uint32_t w) {
    const uint32_t at = Lay::lane(l, w);
    const T* p = X + net_addr<T>(at);
    constexpr uint32_t regs = 15u << Lay::kLow;
    constexpr uint32_t top = (1u << S) >> 1, flip = top ? top - 1u : 0u;
    const T* q = X + net_addr<T>(at ^ (flip & ~regs));
#pragma unroll
    for (uint32_t r = 0; r < kNetRegs; ++r) {
        const uint32_t i = r << Lay::kLow;
        m[r] = i & top ? q[net_addr<T>(i ^ (flip & regs))] : p[net_addr<T>(i)];
        net_single<T>();
    }
}

// ---- stages ---------------------------------------------------------------------
// Register bits HI .. LO, two at a time.
template <class Wd, int HI, int LO>
__device__ __forceinline__ void net_regs(typename Wd::T (&m)[kNetRegs]) {
    if constexpr (HI == LO) {
        constexpr int h = 1 << HI;
#pragma unroll
        for (int e = 0; e < kNetRegs; ++e)
            if (!(e & h)) Wd::cex(m[e], m[e | h]);
    } else if constexpr (HI > LO) {
        constexpr int h = 1 << HI, l = h / 2;
#pragma unroll
        for (int e = 0; e < kNetRegs; ++e)
            if (!(e & (h | l))) Wd::cex4(m[e], m[e | l], m[e | h], m[e | h | l]);
        net_regs<Wd, HI - 2, LO>(m);
    }
}

// One stage across lanes (CTRL: quad_perm to the lane XOR 1, 2 or 3); a mirror
// stage meets the other lane's registers in reverse.  A DPP read needs two
// wait states after its register was written, and the compiler does not count
// the writes of inline assembly.
template <class Wd, int CTRL, bool MIRROR>
__device__ __forceinline__ void net_lanes(typename Wd::T (&m)[kNetRegs], bool upper) {
#pragma unroll
    for (int e = 0; e < kNetRegs; e += 8)
        asm("s_nop 1"
            : "+v"(m[e]), "+v"(m[e + 1]), "+v"(m[e + 2]), "+v"(m[e + 3]), "+v"(m[e + 4]), "+v"(m[e + 5]),
              "+v"(m[e + 6]), "+v"(m[e + 7]));
    typename Wd::T o[kNetRegs];
#pragma unroll
    for (int e = 0; e < kNetRegs; ++e) o[e] = Wd::template dpp<CTRL>(m[MIRROR ? kNetRegs - 1 - e : e]);
    Wd::keep(m, o, upper);
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kXor3 = 0x1B;   // quad_perm controls

// Steps 1 .. 4: sort a lane's words.
template <class Wd, int S>
__device__ __forceinline__ void net_reg_step(typename Wd::T (&m)[kNetRegs]) {
    constexpr int n = 1 << S;
#pragma unroll
    for (int b = 0; b < kNetRegs; b += n) {   // the upper half in reverse: a bitonic sequence
#pragma unroll
        for (int e = 0; e < n / 4; ++e) {
            const typename Wd::T t = m[b + n / 2 + e];
            m[b + n / 2 + e] = m[b + n - 1 - e];
            m[b + n - 1 - e] = t;
        }
    }
    net_regs<Wd, S - 1, 0>(m);
}

// Steps 7 .. 10.
template <class Wd, int S>
__device__ __forceinline__ void net_wave_step(typename Wd::T* X, typename Wd::T (&m)[kNetRegs], uint32_t l, uint32_t w) {
    using T = typename Wd::T;
    net_put<NetA<T>>(X, m, l, w);
    lds_wave_sync();
    net_get<NetB<T, S>, S>(X, m, l, w);
    lds_wave_sync();
    net_regs<Wd, 3, 0>(m);          // index bits S-1 .. S-4
    net_put<NetB<T, S>>(X, m, l, w);
    lds_wave_sync();
    net_get<NetA<T>, 0>(X, m, l, w);
    lds_wave_sync();
    if constexpr (S > 9) net_lanes<Wd, kXor2, false>(m, (l & 2u) != 0);
    if constexpr (S > 8) net_lanes<Wd, kXor1, false>(m, (l & 1u) != 0);
    net_regs<Wd, S < 8 ? S - 5 : 3, 0>(m);
}

// Steps 11 .. 13, the whole workgroup.
template <class Wd, int S>
__device__ __forceinline__ void net_tile_step(typename Wd::T* X, typename Wd::T (&m)[kNetRegs], uint32_t l, uint32_t w) {
    using T = typename Wd::T;
    net_put<NetA<T>>(X, m, l, w);      // the wave read these places last
    lds_barrier();
    net_get<NetC<T, S>, S>(X, m, l, w);
    net_regs<Wd, 3, 0>(m);          // index bits S-1 .. S-4
    lds_barrier();                  // mirrored reads took other waves' places
    net_put<NetC<T, S>>(X, m, l, w);   // C and D: the same places of each wave
    lds_wave_sync();
    net_get<NetD<T, S>, 0>(X, m, l, w);
    lds_wave_sync();
    net_regs<Wd, 3, 0>(m);          // index bits S-5 .. S-8
    net_put<NetD<T, S>>(X, m, l, w);
    lds_barrier();
    net_get<NetA<T>, 0>(X, m, l, w);
    lds_wave_sync();
    if constexpr (S > 12) net_lanes<Wd, kXor1, false>(m, (l & 1u) != 0);
    net_regs<Wd, S < 12 ? S - 9 : 3, 0>(m);
}

// Sort the tile's 1024*W words, of which the first cnt are not sentinels; the
// input may be in any order (registers past cnt hold sentinels), the result is
// left in layout A.  X: net_words<T>(1024*W) words of LDS.  A wave of sentinels
// does nothing, and a step that only brings in sentinels is left out.
template <class Wd, int W>
__device__ __forceinline__ void net_sort(typename Wd::T* X, typename Wd::T (&m)[kNetRegs], uint32_t cnt, int lane,
                                         int wave) {
    static_assert(W == 1 || W == 2 || W == 4 || W == 8, "whole wave bits");
    const uint32_t l = (uint32_t)lane, w = (uint32_t)wave;
    if (w * 1024u < cnt) {
        net_reg_step<Wd, 1>(m);
        net_reg_step<Wd, 2>(m);
        net_reg_step<Wd, 3>(m);
        net_reg_step<Wd, 4>(m);
        net_lanes<Wd, kXor1, true>(m, (l & 1u) != 0);
        net_regs<Wd, 3, 0>(m);
        net_lanes<Wd, kXor3, true>(m, (l & 2u) != 0);
        net_lanes<Wd, kXor1, false>(m, (l & 1u) != 0);
        net_regs<Wd, 3, 0>(m);
        net_wave_step<Wd, 7>(X, m, l, w);
        net_wave_step<Wd, 8>(X, m, l, w);
        net_wave_step<Wd, 9>(X, m, l, w);
        net_wave_step<Wd, 10>(X, m, l, w);
    }
    if constexpr (W >= 2)
        if (cnt > 1024u) net_tile_step<Wd, 11>(X, m, l, w);
    if constexpr (W >= 4)
        if (cnt > 2048u) net_tile_step<Wd, 12>(X, m, l, w);
    if constexpr (W >= 8)
        if (cnt > 4096u) net_tile_step<Wd, 13>(X, m, l, w);
}

// From layout A to the order of memory, inside the wave: register 4c + q of
// lane l holds word 256c + 4l + q of its wave's 1024.
template <class T>
__device__ __forceinline__ void net_to_memory_order(T* X, T (&m)[kNetRegs], uint32_t l, uint32_t w) {
    net_put<NetA<T>>(X, m, l, w);
    lds_wave_sync();
    const T* p = X + net_addr<T>((w << 10) | (l << 2));
#pragma unroll
    for (uint32_t r = 0; r < kNetRegs; ++r) {
        m[r] = p[net_addr<T>(256u * (r >> 2) + (r & 3u))];
        net_single<T>();
    }
    lds_wave_sync();
}

}  // namespace mms
