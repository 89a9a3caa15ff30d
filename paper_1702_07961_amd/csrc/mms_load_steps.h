// How a merge workgroup's waves share the loads of a tile's pieces.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mms_tile_plan.h"

namespace mms {

// Pieces are loaded in steps of 2^S elements of one piece.  Step e of the tile
// sits in lane e of every wave: where its elements come from (in the group),
// its first LDS slot and its length.  Wave w takes steps w, w + W, ...
struct LoadSteps {
    uint32_t src, dst, cnt, total;
};
template <uint32_t S>
__device__ __forceinline__ LoadSteps load_steps(const PieceLayout& pc, uint32_t s, uint32_t Kg, uint64_t L, int lane) {
    const uint32_t own = (pc.len + (1u << S) - 1u) >> S;   // lanes k < Kg hold piece k, the others none
    const uint32_t before = excl_scan16(own);
    // pieces whose steps end at or before this lane's: of the sorted ends (16 at
    // most), how many of every fourth, then how many of the three up to the next
    const uint32_t end = before + own;
    uint32_t k = 0;
#pragma unroll
    for (int j = 3; j < 15; j += 4) k += (uint32_t)__builtin_amdgcn_readlane((int)end, j) <= (uint32_t)lane ? 4u : 0u;
    const int k4 = (int)(k << 2);
    const uint32_t e0 = (uint32_t)__builtin_amdgcn_ds_bpermute(k4, (int)end);
    const uint32_t e1 = (uint32_t)__builtin_amdgcn_ds_bpermute(k4 + 4, (int)end);
    const uint32_t e2 = (uint32_t)__builtin_amdgcn_ds_bpermute(k4 + 8, (int)end);
    k += (e0 <= (uint32_t)lane ? 1u : 0u) + (e1 <= (uint32_t)lane ? 1u : 0u) + (e2 <= (uint32_t)lane ? 1u : 0u);
    const uint32_t from = (uint32_t)((uint64_t)(uint32_t)lane * L) + s;   // lane k: piece k's first element
    auto of = [&](uint32_t x) { return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(k << 2), (int)x); };
    const uint32_t at = ((uint32_t)lane - of(before)) << S;
    LoadSteps r;
    r.src = of(from) + at;
    r.dst = of(pc.sb) + at;
    r.cnt = min(of(pc.len) - at, 1u << S);   // meaningful below total only
    r.total = (uint32_t)__builtin_amdgcn_readlane((int)end, 15);
    return r;
}

}  // namespace mms
