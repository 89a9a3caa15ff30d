// The block step of the keys merge: 16 lanes (one DPP row) merge 16*EM
// outputs of a pair of runs held in LDS.
//
// Work is planned in items: an item is up to 4*(4*EM - 2) consecutive outputs
// of one pair of runs, and every row of a workgroup takes one item of a merge
// level at a time.  Slots, run bounds and output offsets are multiples of 4,
// so all of them are counted in 16-byte chunks, and every LDS access of a
// block is one 128-bit access per lane at consecutive chunks.  Runs end on a
// chunk boundary: the slots past a piece's last key hold the largest key, so
// those keys sort to the tile's end, past its last real output.
//
// Why rows: a block of 16*EM keys (EM per lane) needs log2(16*EM) stages
// whatever its lanes, so 256-key blocks of one row (16 per lane) take two
// stages fewer than 1024-key blocks of a wave, every lane distance is a DPP
// exchange, and a 16-lane search finds the split in two or three rounds.
// One 128-bit read takes 1.1 LDS cycles per 64 keys where 64 consecutive
// words take 2.3, and writes cost three times as much (3.4), so a block reads
// and writes LDS once in 16-byte chunks and moves only two index bits through
// scratch: merge launch of 10^8 keys 0.326 ms with all lane bits by DPP, 0.303
// with bits 5 and 4 through scratch, 0.348 with bits 3 and 2 as well (its
// stores then conflict four ways); the probe spread below took it to 0.297.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "mms_device.h"
#include "mms_tile_plan.h"

namespace mms {

// Compare-exchange of lanes 4 apart in their row: the lower one keeps the
// minimum, the upper one the maximum, each in one instruction that writes
// only the 4-lane banks it concerns.  (A DPP read needs two wait states after
// the register was written, which the leading s_nop provides.)
__device__ __forceinline__ void lane4_cex(uint32_t& a, uint32_t& b, uint32_t& c, uint32_t& d) {
    uint32_t x, y, z, w;
    asm("s_nop 1\n\t"
        "v_min_u32_dpp %0, %4, %4 row_shl:4 row_mask:0xf bank_mask:0x5\n\t"
        "v_min_u32_dpp %1, %5, %5 row_shl:4 row_mask:0xf bank_mask:0x5\n\t"
        "v_min_u32_dpp %2, %6, %6 row_shl:4 row_mask:0xf bank_mask:0x5\n\t"
        "v_min_u32_dpp %3, %7, %7 row_shl:4 row_mask:0xf bank_mask:0x5\n\t"
        "v_max_u32_dpp %0, %4, %4 row_shr:4 row_mask:0xf bank_mask:0xa\n\t"
        "v_max_u32_dpp %1, %5, %5 row_shr:4 row_mask:0xf bank_mask:0xa\n\t"
        "v_max_u32_dpp %2, %6, %6 row_shr:4 row_mask:0xf bank_mask:0xa\n\t"
        "v_max_u32_dpp %3, %7, %7 row_shr:4 row_mask:0xf bank_mask:0xa"
        : "=&v"(x), "=&v"(y), "=&v"(z), "=&v"(w)
        : "v"(a), "v"(b), "v"(c), "v"(d));
    a = x;
    b = y;
    c = z;
    d = w;
}

// Words of a wave's transpose scratch: four rows of 64, four words apart in
// the banks.
constexpr uint32_t kRowXposeStride = 68;
constexpr uint32_t kRowXposeWords = 4u * kRowXposeStride;

// Sort the bitonic sequence of 16*EM keys a row holds, key 4c + j of lane i
// being position 64c + 4i + j.  Index bits above 5 are register bits, then
// bits 5 and 4 (lane bits 3 and 2) change places with register bits 7 and 6
// through the wave's scratch (EM = 16), bits 3 and 2 meet across lanes and
// bits 1 and 0 are in the chunk.  The result is left with chunk c of lane i at
// chunk row_chunk0<EM>(i) + kRowChunkStep<EM> * c of the sorted sequence.
template <int EM>
__device__ __forceinline__ uint32_t row_chunk0(uint32_t i) {
    return EM == 16 ? 16u * (i >> 2) + (i & 3u) : i;
}
template <int EM> constexpr uint32_t kRowChunkStep = EM == 16 ? 4u : 16u;

template <int EM>
__device__ __forceinline__ void row_sort(uint32_t (&m)[EM], uint32_t* scr, int lane) {
    static_assert(EM == 8 || EM == 16, "two or four chunks per lane");
    auto lane_stage = [&](auto ctrl, int dist) {
        const uint32_t keep = (lane & dist) ? ~0u : 0u;
        uint32_t o[EM];   // all exchanges first: no wait states between a write and its exchange
#pragma unroll
        for (int e = 0; e < EM; ++e)
            o[e] = (uint32_t)__builtin_amdgcn_mov_dpp((int)m[e], decltype(ctrl)::value, 0xF, 0xF, false);
#pragma unroll
        for (int e = 0; e < EM; ++e) m[e] = med3_u32(m[e], o[e], keep);
    };
    if constexpr (EM == 16) {
        const uint32_t ul = (uint32_t)lane;
        uint32_t* rd = scr + ((ul >> 2) & 3u) * kRowXposeStride + (ul & 48u) + (ul & 3u);
        asm volatile("" ::: "memory");      // the previous block's scratch reads come first
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            bitonic4(m[j], m[4 + j], m[8 + j], m[12 + j]);
#pragma unroll
            for (uint32_t c = 0; c < 4u; ++c) scr[c * kRowXposeStride + ul] = m[4 * c + j];
            lds_wave_sync();
#pragma unroll
            for (uint32_t c = 0; c < 4u; ++c) m[4 * c + j] = rd[4u * c];
            lds_wave_sync();
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) bitonic4(m[j], m[4 + j], m[8 + j], m[12 + j]);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) cex_u32(m[j], m[4 + j]);
        lane_stage(std::integral_constant<int, 0x128>{}, 8);    // row_ror:8
#pragma unroll
        for (int c = 0; c < EM / 4; ++c) lane4_cex(m[4 * c], m[4 * c + 1], m[4 * c + 2], m[4 * c + 3]);
    }
    lane_stage(std::integral_constant<int, 0x4E>{}, 2);     // quad_perm [2,3,0,1]
    lane_stage(std::integral_constant<int, 0xB1>{}, 1);     // quad_perm [1,0,3,2]
#pragma unroll
    for (int c = 0; c < EM / 4; ++c) bitonic4(m[4 * c], m[4 * c + 1], m[4 * c + 2], m[4 * c + 3]);
}

// ---- items --------------------------------------------------------------------
// Outputs of one item at most, in chunks: a block's 16*EM keys less two chunks,
// which the block may spend on outputs of the item before it.
template <int EM> constexpr uint32_t kItemChunks = 4u * EM - 2u;

template <int EM, int W, uint32_t TMAX>
struct RowItems {
    static constexpr uint32_t kChunks = TMAX / 4u + kMaxFanout;   // LDS slots of a tile
    static constexpr uint32_t kRows = 4u * W;
    // a pair's last item may be partial
    static constexpr uint32_t kPerLevel = kChunks / kItemChunks<EM> + kMaxFanout / 2u;
    static constexpr uint32_t kWords = 4u * kPerLevel * 2u + 16u;
    static_assert(kChunks < 4096u, "chunk numbers take 12 bits");
    static_assert((kChunks + kItemChunks<EM> - 1u) / kItemChunks<EM> <= kRows, "a pass holds any pair");

    __device__ static __forceinline__ void build(uint32_t* items, const uint32_t* sbeg, uint32_t Kg, int lane) {
        build_items<2, kItemChunks<EM>, kPerLevel>(items, sbeg, Kg, lane);
    }
};

// ---- one item -------------------------------------------------------------------
struct RowOut {
    uint32_t chunk;   // first output chunk of the item (of the tile's slots)
    uint32_t pad;     // leading chunks of the block that belong to the item before (0 to 2)
    uint32_t cnt;     // chunks of the item (0: none)
};

// Merge one item per row: X holds the level's runs, w the item's words;
// the block is left sorted in m (layout of row_sort).
//
// The split of the pair at the item's first output d0 is searched in chunks
// only, 16 lanes probing per round (a range of up to 15 chunks takes one
// round, 255 two): T = the number of chunks c of A whose key 4c + r precedes
// B's key 4 d0 - 1 - (4c + r), so A holds more than 4(T-1) + r and at most
// 4T + r of the pair's first 4 d0 outputs.  r is the row's number: keys at
// multiples of four lie in 8 of the 32 banks only, so the rows probe next to
// each other, and an odd distance between probes visits all 8.  A block that
// starts at chunk T-1 of A and d0 - T - 1 of B (not below 0) begins inside
// both runs' share of those outputs and takes in at most two chunks' worth of
// them, which are no larger than any other key of the block: they sort to its
// front and are not stored.
//
// lone: some pairs may have one run only, and this is not the last level.  A
// wave whose items are all of such pairs leaves them where they are, which
// their outputs' slots are too: 10^8 nearly sorted keys (10^6 swaps) 1453 ->
// 1358 us, sorted 1460 -> 1255.  Asked with 256-key blocks only: launches of
// the smaller ones are short of latency, not of issue (2^20 keys 65.4 -> 66.0).
template <int EM>
__device__ __forceinline__ RowOut row_merge(const uint32_t* X, uint2 w, const uint32_t* sent, uint32_t* scr,
                                            uint32_t (&m)[EM], int lane, bool lone) {
    const uint32_t i = (uint32_t)lane & 15u, row = (uint32_t)lane >> 4;
    const uint32_t aA = w.x & 0xFFFu, aB = w.x >> 12;
    const uint32_t d0 = (w.y >> 12) & 0xFFFu, en = w.y & 0xFFFu;
    const uint32_t la = aB - aA, lb = en - aB;
    if constexpr (EM == 16) {
        if (lone && __ballot(la != 0u && lb != 0u) == 0ull) {
#pragma unroll
            for (int e = 0; e < EM; ++e) asm("" : "=v"(m[e]));     // not stored, whatever they hold
            return RowOut{0, 0, 0};
        }
    }
    uint32_t lo = d0 > lb ? d0 - lb : 0u;
    uint32_t hi = min(d0, la);
    // A lane past the range probes up to 31 chunks past it (inside the
    // workgroup's LDS: the layout keeps that much before and after the keys)
    // and does not count; at most 15 probes precede the split.
    const uint32_t* pA = X + (4u * aA + row);
    const uint32_t* pB = X + (4u * (aB + d0) - 1u - row);
    while (__ballot(lo < hi)) {
        // probes s + 1 chunks apart, an odd number (below): bank spread
        const uint32_t s = (((hi - lo) >> 4) + 1u) & ~1u;
        const uint32_t c = lo + i + __umul24(s, i + 1u);
        const bool before = pA[4u * c] <= *(pB - 4u * c);
        const uint64_t bal = __ballot(c < hi) & __ballot(before);
        const uint32_t t = (uint32_t)__popc((uint32_t)(bal >> ((uint32_t)lane & 48u)) & 0xFFFFu);
        lo += __umul24(t, s) + t;
        hi = min(hi, lo + s);
    }
    const uint32_t T = lo;
    // first chunks of the block in A and in B
    const uint32_t p = T ? T - 1u : 0u, q = d0 > T ? d0 - T - 1u : 0u;
    const uint32_t pad = d0 - p - q;
    uint32_t a[EM], b[EM];
    constexpr uint32_t Q = EM / 4;            // chunks per lane
    auto get = [&](uint32_t (&r)[EM], int c, const uint32_t* from, bool rev) {
        const uint4 v = *reinterpret_cast<const uint4*>(from);
        r[4 * c + 0] = rev ? v.w : v.x;
        r[4 * c + 1] = rev ? v.z : v.y;
        r[4 * c + 2] = rev ? v.y : v.z;
        r[4 * c + 3] = rev ? v.x : v.w;
    };
    const uint32_t* Ap = X + 4u * (aA + p + i);
    const uint32_t* Bp = X + 4u * (aB + q + 15u - i);
    if (__ballot(p + 16u * Q > la || q + 16u * Q > lb) == 0ull) {
#pragma unroll
        for (int c = 0; c < (int)Q; ++c) {
            get(a, c, Ap + 64u * (uint32_t)c, false);
            get(b, c, Bp + 64u * (Q - 1u - (uint32_t)c), true);
        }
    } else {
        // chunks past a run's end read the largest key; its address takes each
        // read's offset off, so the offsets stay in the instructions
        const int ra = (int)(la - p - i), rb = (int)(lb - q) - (int)(15u - i);   // chunks from the lane's first on
#pragma unroll
        for (int c = 0; c < (int)Q; ++c) {
            get(a, c, (16 * c < ra ? Ap : sent - 64 * c) + 64 * c, false);
            const int cb = (int)Q - 1 - c;
            get(b, c, (16 * cb < rb ? Bp : sent - 64 * cb) + 64 * cb, true);
        }
    }
#pragma unroll
    for (int e = 0; e < EM; ++e) m[e] = min(a[e], b[e]);
    row_sort<EM>(m, scr, lane);
    return RowOut{aA + d0, pad, w.y >> 24};
}

// The outputs of a sorted item: put(the lane's first chunk, a step from it that
// is a constant, four keys).
template <int EM, class Put>
__device__ __forceinline__ void row_put(const RowOut& o, const uint32_t (&m)[EM], int lane, const Put& put) {
    const uint32_t t0 = row_chunk0<EM>((uint32_t)lane & 15u) - o.pad;   // wraps for the chunks not stored
#pragma unroll
    for (int c = 0; c < EM / 4; ++c) {
        const uint32_t step = kRowChunkStep<EM> * (uint32_t)c;
        if (t0 + step < o.cnt) put((int)(o.chunk + t0), (int)step, m[4 * c], m[4 * c + 1], m[4 * c + 2], m[4 * c + 3]);
    }
}
template <int EM>
__device__ __forceinline__ void row_put_lds(uint32_t* X, const RowOut& o, const uint32_t (&m)[EM], int lane) {
    row_put(o, m, lane, [&](int c, int step, uint32_t k0, uint32_t k1, uint32_t k2, uint32_t k3) {
        *reinterpret_cast<uint4*>(X + 4 * c + 4 * step) = make_uint4(k0, k1, k2, k3);
    });
}

// One merge level in place: the rows of a pass read and sort one item each,
// the workgroup meets, and the items go back to their pairs' slots.  A pass
// takes as many whole pairs as it has rows for (nearly always all), so it
// writes no slot that a later one reads.  The level's last pass leaves its
// items in m and o (o.cnt = 0: none) instead, after the meeting.
template <int EM, class Items>
__device__ __forceinline__ void row_merge_level(uint32_t* X, const uint32_t* items, uint32_t lvl, const uint32_t* sent,
                                                uint32_t* scr, int wave, int lane, bool lone, uint32_t (&m)[EM],
                                                RowOut& o) {
    const uint32_t pairs = 8u >> lvl;
    const uint32_t upto = items[8u * Items::kPerLevel + min(16u - 2u * pairs + (uint32_t)lane, 14u)];
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)upto, (int)(pairs - 1u));
    for (uint32_t beg = 0;;) {
        const uint64_t fit = __ballot((uint32_t)lane < pairs && upto <= beg + Items::kRows);
        const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)upto, __popcll(fit) - 1);
        const uint32_t at = beg + 4u * (uint32_t)wave;   // the wave's first item
        o = RowOut{0, 0, 0};
        if (at < end) {
            const uint32_t it = at + ((uint32_t)lane >> 4);
            uint2 w = *reinterpret_cast<const uint2*>(items + 2u * (lvl * Items::kPerLevel + it));
            if (it >= end) w = make_uint2(0u, 0u);
            o = row_merge<EM>(X, w, sent, scr, m, lane, lone);
        }
        lds_barrier();   // the pass's reads are done
        if (end >= total) break;
        row_put_lds(X, o, m, lane);
        beg = end;
    }
}

}  // namespace mms
