// Row merge of 64-bit words: the block step of the key-value and 64-bit
// merges.  16 lanes (one DPP row) merge 256 (or 128) words of a pair of
// runs in LDS, as the keys merge does with 32-bit keys (mms_row_merge.h).
//
// A word is a positive normal double (mms_device_kt.h) whose mantissa is the
// element's order: the key or its leading bits, then the element's slot in
// the tile as loaded, so words are unique and their order is the stable one.
// v_min_f64 and v_max_f64 run at the rate of the 32-bit ones, so a compare-
// exchange of words costs two instructions.
//
// Work is planned in items, an item being up to 252 (124) consecutive outputs
// of one pair of runs.  Everything is counted in chunks of two words (16 bytes):
// runs start and end on chunks (the slots past a piece hold the sentinel), so
// every LDS access of a block is one 128-bit access per lane at consecutive
// chunks.  A wave's four rows start wherever their items do, so they may meet in
// the banks: 23 to 27 % of the pair merge's LDS cycles, by input.
// A level is merged in place: every row reads its item into registers, the
// workgroup meets, and the sorted items go back to the slots they came from.
// One buffer instead of two is what lets four workgroups share a compute
// unit.
//
// Two of the four lane distances change places with register bits through the
// wave's scratch, a word's halves one after the other, and two are exchanged
// by DPP (two moves for the halves) with one v_min_f64 or v_max_f64 under the
// lanes' mask: four VALU instructions a word against one in a register.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mms_device.h"
#include "mms_device_kt.h"
#include "mms_tile_plan.h"

namespace mms {

// Words of a block per lane: 16 or 8 (256- or 128-word blocks).  Outputs of an
// item at most, in chunks: a block's 16*EM words less two chunks, which the
// block may spend on outputs of the item before it.
template <int EM> constexpr uint32_t kWordItemChunks = 8u * EM - 2u;

// ---- items --------------------------------------------------------------------
template <int EM, uint32_t TOUT, int W>
struct WordItems {
    static constexpr uint32_t kCap = TOUT + 4u * kMaxFanout;    // LDS slots of a tile
    static constexpr uint32_t kRows = 4u * W;
    // a level's pairs hold kCap / 2 chunks in all, and each may end in a
    // partial item
    static constexpr uint32_t kPerLevel = kCap / 2u / kWordItemChunks<EM> + kMaxFanout / 2u;
    static constexpr uint32_t kWords = 4u * kPerLevel * 2u + 16u;
    static_assert(kCap / 2u < 4096u, "chunk numbers take 12 bits");
    static_assert((kCap / 2u + kWordItemChunks<EM> - 1u) / kWordItemChunks<EM> <= kRows, "a pass holds any pair");

    __device__ static __forceinline__ void build(uint32_t* items, const uint32_t* sbeg, uint32_t Kg, int lane) {
        build_items<1, kWordItemChunks<EM>, kPerLevel>(items, sbeg, Kg, lane);
    }
};

// ---- one item -------------------------------------------------------------------
// Compare-exchange of lanes met by a DPP control; the upper lane of each two
// keeps the larger words.  A DPP read needs two wait states after its register
// was written, and the compiler does not count the writes of inline assembly.
template <int CTRL, int EM>
__device__ __forceinline__ void word_lane_stage(double (&m)[EM], bool upper) {
#pragma unroll
    for (int e = 0; e < EM; e += 8)
        asm("s_nop 1"
            : "+v"(m[e]), "+v"(m[e + 1]), "+v"(m[e + 2]), "+v"(m[e + 3]), "+v"(m[e + 4]), "+v"(m[e + 5]),
              "+v"(m[e + 6]), "+v"(m[e + 7]));
    double o[EM];
#pragma unroll
    for (int e = 0; e < EM; ++e)
        o[e] = kt_join((uint32_t)__builtin_amdgcn_mov_dpp((int)kt_hi(m[e]), CTRL, 0xF, 0xF, false),
                       (uint32_t)__builtin_amdgcn_mov_dpp((int)kt_lo(m[e]), CTRL, 0xF, 0xF, false));
    if (upper) {
#pragma unroll
        for (int e = 0; e < EM; ++e) m[e] = kt_max(m[e], o[e]);
    } else {
#pragma unroll
        for (int e = 0; e < EM; ++e) m[e] = kt_min(m[e], o[e]);
    }
}

// Words of a wave's transpose scratch: four rows of 64 half words, four words
// apart in the banks.
constexpr uint32_t kWordXposeStride = 68;
constexpr uint32_t kWordXposeWords = 4u * kWordXposeStride;

// Sort the bitonic sequence of 16*EM words a row holds, word 2c + j of lane i
// being position 32c + 2i + j.  Index bits above 4 are register bits; then
// bits 4 and 3 (lane bits 3 and 2) change places with the top two register
// bits through the scratch, bits 2 and 1 meet across lanes and bit 0 is in the
// chunk.  Words e, e + 1 of lane i (e even) are left at chunk
// word_chunk0<EM>(i) + word_step<EM>(e) of the sorted sequence.
template <int EM>
__device__ __forceinline__ uint32_t word_chunk0(uint32_t i) {
    return 2u * EM * (i >> 2) + (i & 3u);
}
template <int EM>
__device__ __forceinline__ constexpr uint32_t word_step(uint32_t e) {
    constexpr uint32_t G = EM / 4;   // words per value of the exchanged bits
    return 4u * (e / G) + 16u * (e % G / 2u);
}

template <int EM>
__device__ __forceinline__ void word_row_sort(double (&m)[EM], uint32_t* scr, int lane) {
    static_assert(EM == 8 || EM == 16, "four or eight chunks per lane");
    constexpr int G = EM / 4;
    const uint32_t ul = (uint32_t)lane;
    uint32_t* wr = scr + ul;
    const uint32_t* rd = scr + ((ul >> 2) & 3u) * kWordXposeStride + (ul & 48u) + (ul & 3u);
    asm volatile("" ::: "memory");      // the previous block's scratch reads come first
#pragma unroll
    for (int d = EM / 2; d >= 2; d >>= 1) {
#pragma unroll
        for (int e = 0; e < EM; ++e)
            if ((e & d) == 0) cex_kt(m[e], m[e | d]);
    }
#pragma unroll
    for (int x = 0; x < G; ++x) {
        uint32_t h[4], l[4];
#pragma unroll
        for (uint32_t g = 0; g < 4u; ++g) wr[g * kWordXposeStride] = kt_hi(m[G * g + x]);
        lds_wave_sync();
#pragma unroll
        for (uint32_t g = 0; g < 4u; ++g) h[g] = rd[4u * g];
        lds_wave_sync();
#pragma unroll
        for (uint32_t g = 0; g < 4u; ++g) wr[g * kWordXposeStride] = kt_lo(m[G * g + x]);
        lds_wave_sync();
#pragma unroll
        for (uint32_t g = 0; g < 4u; ++g) l[g] = rd[4u * g];
        lds_wave_sync();
#pragma unroll
        for (uint32_t g = 0; g < 4u; ++g) m[G * g + x] = kt_join(h[g], l[g]);
    }
#pragma unroll
    for (int d = EM / 2; d >= G; d >>= 1) {
#pragma unroll
        for (int e = 0; e < EM; ++e)
            if ((e & d) == 0) cex_kt(m[e], m[e | d]);
    }
    word_lane_stage<0x4E, EM>(m, (ul & 2u) != 0);           // quad_perm [2,3,0,1]
    word_lane_stage<0xB1, EM>(m, (ul & 1u) != 0);           // quad_perm [1,0,3,2]
#pragma unroll
    for (int e = 0; e < EM; e += 2) cex_kt(m[e], m[e + 1]);
}

struct WordRow {
    uint32_t chunk;   // first output chunk of the item (of the tile's slots)
    uint32_t pad;     // leading chunks of the block that belong to the item before (0 to 2)
    uint32_t cnt;     // chunks of the item (0: none)
};

// Merge one item per row: X holds the level's runs, w the item's words; the
// block is left sorted in m (layout of word_row_sort).
//
// The split of the pair at the item's first output d0 is searched in chunks
// only, 16 lanes probing per round: T = the number of chunks c of A whose
// word 2c + r precedes B's word 2 d0 - 1 - (2c + r), r being 0 or 1 by the
// row's number (the rows then probe different banks).  A holds more than
// 2(T-1) + r and at most 2T + r of the pair's first 2 d0 outputs, so a block
// that starts at chunk T-1 of A and d0 - T - 1 of B (not below 0) begins
// inside both runs' share of them and takes in at most two chunks' worth,
// which are no larger than any other word of the block: they sort to its
// front and are not stored.
template <int EM>
__device__ __forceinline__ WordRow word_row_merge(const double* X, uint2 w, const double* sent, uint32_t* scr,
                                                  double (&m)[EM], int lane) {
    const uint32_t i = (uint32_t)lane & 15u, r = ((uint32_t)lane >> 4) & 1u;
    const uint32_t aA = w.x & 0xFFFu, aB = w.x >> 12;
    const uint32_t d0 = (w.y >> 12) & 0xFFFu, en = w.y & 0xFFFu;
    const uint32_t la = aB - aA, lb = en - aB;
    uint32_t lo = d0 > lb ? d0 - lb : 0u;
    uint32_t hi = min(d0, la);
    // a lane past the range probes up to 31 chunks past it (inside the
    // workgroup's LDS: the layout keeps that much around the words) and does
    // not count; at most 15 probes precede the split
    const double* pA = X + (2u * aA + r);
    const double* pB = X + (2u * (aB + d0) - 1u - r);
    while (__ballot(lo < hi)) {
        // probes s + 1 chunks apart, an odd number: bank spread
        const uint32_t s = (((hi - lo) >> 4) + 1u) & ~1u;
        const uint32_t c = lo + i + __umul24(s, i + 1u);
        const bool before = pA[2u * c] <= *(pB - 2u * c);
        const uint64_t bal = __ballot(c < hi) & __ballot(before);
        const uint32_t t = (uint32_t)__popc((uint32_t)(bal >> ((uint32_t)lane & 48u)) & 0xFFFFu);
        lo += __umul24(t, s) + t;
        hi = min(hi, lo + s);
    }
    const uint32_t T = lo;
    const uint32_t p = T ? T - 1u : 0u, q = d0 > T ? d0 - T - 1u : 0u;
    constexpr uint32_t Q = EM / 2;   // chunks per lane
    typedef double d2 __attribute__((ext_vector_type(2)));
    const double* Ap = X + 2u * (aA + p + i);
    const double* Bp = X + 2u * (aB + q + 15u - i);
    if (__ballot(p + 16u * Q > la || q + 16u * Q > lb) == 0ull) {
#pragma unroll
        for (uint32_t c = 0; c < Q; ++c) {
            const d2 a = *reinterpret_cast<const d2*>(Ap + 32u * c);
            const d2 b = *reinterpret_cast<const d2*>(Bp + 32u * (Q - 1u - c));
            m[2 * c] = kt_min(a.x, b.y);
            m[2 * c + 1] = kt_min(a.y, b.x);
        }
    } else {
        // chunks past a run's end read the sentinel; its address takes each
        // read's offset off, so the offsets stay in the instructions
        const int ra = (int)(la - p - i), rb = (int)(lb - q) - (int)(15u - i);   // chunks from the lane's first on
#pragma unroll
        for (int c = 0; c < (int)Q; ++c) {
            const int cb = (int)Q - 1 - c;
            const double* from_a = 16 * c < ra ? Ap : sent - 32 * c;
            const double* from_b = 16 * cb < rb ? Bp : sent - 32 * cb;
            const d2 a = *reinterpret_cast<const d2*>(from_a + 32 * c);
            const d2 b = *reinterpret_cast<const d2*>(from_b + 32 * cb);
            m[2 * c] = kt_min(a.x, b.y);
            m[2 * c + 1] = kt_min(a.y, b.x);
        }
    }
    word_row_sort<EM>(m, scr, lane);
    return WordRow{aA + d0, d0 - p - q, w.y >> 24};
}

// The outputs of a sorted item: put(the lane's first chunk, a step from it that
// is a constant, word, word).
template <int EM, class Put>
__device__ __forceinline__ void word_row_put(const WordRow& o, const double (&m)[EM], int lane, const Put& put) {
    const uint32_t t0 = word_chunk0<EM>((uint32_t)lane & 15u) - o.pad;   // wraps for the chunks not stored
#pragma unroll
    for (int e = 0; e < EM; e += 2) {
        const uint32_t step = word_step<EM>((uint32_t)e);
        if (t0 + step < o.cnt) put((int)(o.chunk + t0), (int)step, m[e], m[e + 1]);
    }
}
template <int EM>
__device__ __forceinline__ void word_put_lds(double* X, const WordRow& o, const double (&m)[EM], int lane) {
    typedef double d2 __attribute__((ext_vector_type(2)));
    word_row_put(o, m, lane, [&](int c, int step, double a, double z) {
        *reinterpret_cast<d2*>(X + 2 * c + 2 * step) = d2{a, z};
    });
}

// One merge level in place: the rows of a pass read and sort one item each,
// the workgroup meets, and the items go back to their pairs' slots.  A pass
// takes as many whole pairs as it has rows for (nearly always all), so it
// writes no slot that a later one reads.  The level's last pass leaves its
// items in m and o (o.cnt = 0: none) instead, after the meeting.
template <int EM, class Items>
__device__ __forceinline__ void word_merge_level(double* X, const uint32_t* items, uint32_t lvl, const double* sent,
                                                 uint32_t* scr, int wave, int lane, double (&m)[EM],
                                                 WordRow& o) {
    const uint32_t pairs = 8u >> lvl;
    const uint32_t upto = items[8u * Items::kPerLevel + min(16u - 2u * pairs + (uint32_t)lane, 14u)];
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)upto, (int)(pairs - 1u));
    for (uint32_t beg = 0;;) {
        const uint64_t fit = __ballot((uint32_t)lane < pairs && upto <= beg + Items::kRows);
        const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)upto, __popcll(fit) - 1);
        const uint32_t at = beg + 4u * (uint32_t)wave;   // the wave's first item
        o = WordRow{0, 0, 0};
        if (at < end) {
            const uint32_t it = at + ((uint32_t)lane >> 4);
            uint2 w = *reinterpret_cast<const uint2*>(items + 2u * (lvl * Items::kPerLevel + it));
            if (it >= end) w = make_uint2(0u, 0u);
            o = word_row_merge<EM>(X, w, sent, scr, m, lane);
        }
        lds_barrier();   // the pass's reads are done
        if (end >= total) break;
        word_put_lds(X, o, m, lane);
        beg = end;
    }
}

}  // namespace mms
