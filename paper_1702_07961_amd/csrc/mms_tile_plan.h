// Piece layout of the K-way merges (§4.2): where each run's piece of a merge
// tile sits in LDS.  Shared by the merge kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mms_device.h"
#include "mms_internal.h"

namespace mms {

// Exclusive sum over the 16 lanes of each row (DPP row shifts; a lane
// shifted in from outside the row reads 0).
__device__ __forceinline__ uint32_t excl_scan16(uint32_t x) {
    uint32_t incl = x;
    incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x111, 0xF, 0xF, false);   // row_shr:1
    incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x112, 0xF, 0xF, false);   // row_shr:2
    incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x114, 0xF, 0xF, false);   // row_shr:4
    incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x118, 0xF, 0xF, false);   // row_shr:8
    return incl - x;
}

// Piece layout of a tile of cnt outputs from Kg runs, in registers: lane
// k < Kg, holding run k's split indices s <= e, gets its piece's length and its
// 4-aligned first LDS slot.
struct PieceLayout {
    uint32_t len, sb;
};
__device__ __forceinline__ PieceLayout piece_layout(uint32_t s, uint32_t e, uint32_t Kg, uint32_t cnt, int lane) {
    const bool own = (uint32_t)lane < Kg;
    uint32_t len = own ? e - s : 0u;
    const uint32_t pl = excl_scan16(len);
    // guards for memory safety only: keep the pieces inside the tile
    len = pl >= cnt ? 0u : min(len, cnt - pl);
    const uint32_t sb = excl_scan16((len + 3u) & ~3u);
    return {len, sb};
}

// The items of every merge level of a tile (one wave), in chunks of 2^SHIFT
// slots, each of up to ITEM chunks of outputs of one pair.  Item words: word 0 =
// first chunk of the pair's run A (bits 0..11) and of run B (12..23); word 1 =
// end of run B (0..11), first output of the item inside the pair (12..23),
// outputs (24..31, 0: no item).  After the items (PER_LEVEL for each level),
// for each pair (8, 4, 2 and 1), the items of its level up to its end.
// sbeg: first slots of the pieces, sbeg[Kg] the end.
//
// Lane q < 15 takes pair p of level l (8, 4, 2 and 1 pairs): its runs' bounds
// from the piece starts, the fewest items that hold it, and equal shares.  The
// items are then written by rows, four pairs at a time, a lane each: the wave
// that plans does so while the others wait for it, and its 15 trips of one pair
// took 600 vector instructions, its four trips 120.  With the piece of a load
// step found in one step of four and one of three (mms_load_steps.h) instead
// of 15, sorts of 40,961 keys 26.9 -> 26.1 us, 6.3 million 151.0 -> 146.1, 10^8
// 1601 -> 1566; 2^27 pairs 4399 -> 4277; 10^8 64-bit keys 3954 -> 3850.
template <uint32_t SHIFT, uint32_t ITEM, uint32_t PER_LEVEL>
__device__ __forceinline__ void build_items(uint32_t* items, const uint32_t* sbeg, uint32_t Kg, int lane) {
    const uint32_t q = (uint32_t)lane;
    const uint32_t l = q < 8u ? 0u : q < 12u ? 1u : q < 14u ? 2u : 3u;
    const uint32_t p = q < 8u ? q : q < 12u ? q - 8u : q < 14u ? q - 12u : 0u;
    const uint32_t a = sbeg[min((2u * p) << l, Kg)] >> SHIFT;
    const uint32_t b = sbeg[min((2u * p + 1u) << l, Kg)] >> SHIFT;
    const uint32_t e = sbeg[min((2u * p + 2u) << l, Kg)] >> SHIFT;
    const uint32_t size = q < 15u ? e - a : 0u;
    const uint32_t nit = udiv_small(size + ITEM - 1u, ITEM);
    const uint32_t share = nit ? udiv_small(size + nit - 1u, nit) : 0u;
    // first item of the pair in its level: items of the level's pairs before it
    const uint32_t before = excl_scan16(nit);
    const uint32_t lv0 = l == 0u ? 0u : l == 1u ? 8u : l == 2u ? 12u : 14u;
    const uint32_t first = before - (uint32_t)__builtin_amdgcn_ds_bpermute((int)(lv0 << 2), (int)before);
    if (q < 15u) items[8u * PER_LEVEL + q] = first + nit;
    const uint32_t w0 = a | (b << 12) | (nit << 24), w1 = e | (size << 12) | (share << 24);
    const uint32_t at = l * PER_LEVEL + first;
#pragma unroll 1
    for (uint32_t s = 0; s < 16u; s += 4u) {   // row r: pair s + r (lane 15's has no items)
        const int from = (int)(4u * (s + (q >> 4)));
        const uint32_t r0 = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)w0);
        const uint32_t r1 = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)w1);
        const uint32_t ra = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)at);
        const uint32_t n = r0 >> 24, sh = r1 >> 24, sz = (r1 >> 12) & 0xFFFu;
        for (uint32_t j = q & 15u; j < n; j += 16u) {
            const uint32_t d0 = __umul24(j, sh);
            const uint32_t cnt = sz > d0 ? min(sh, sz - d0) : 0u;
            *reinterpret_cast<uint2*>(items + 2u * (ra + j)) =
                make_uint2(r0 & 0xFFFFFFu, (r1 & 0xFFFu) | (d0 << 12) | (cnt << 24));
        }
    }
}

}  // namespace mms
