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

}  // namespace mms
