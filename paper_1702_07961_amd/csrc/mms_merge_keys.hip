// Keys-only K-way merge round (§4.2, §7), one workgroup per output tile.
//
// A tile's input is the K pieces of its group's runs bounded by the split
// indices of its first and last output (§4.1).  The pieces are loaded to
// 4-aligned offsets of an LDS buffer and merged pairwise, level by level, in
// row blocks (mms_row_merge.h), log2 K levels, in place; the last level stores
// straight from registers to memory.  Nothing is prefetched: with one buffer
// of four bytes a key four workgroups of eight waves share a compute unit, and
// the others merge while one loads.
//
// Bound by VALU issue: it issues in all of the launch's cycles (LDS busy in
// half of them).  10^8 keys, K = 16, 7424-key tiles: 248 us per launch on
// average, 3.2 TB/s; as a persistent kernel of two workgroups per compute unit
// that loaded the next tile into registers and a second buffer meanwhile, 297
// with VALU in 75 % of the cycles.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mms_device.h"
#include "mms_internal.h"
#include "mms_load_steps.h"
#include "mms_row_merge.h"

namespace mms {

// LDS words before the keys (the waves' transpose scratch) and after them (a
// chunk of the largest key, the items, the piece starts).
template <int EM, int W, uint32_t TMAX>
constexpr uint32_t kMergeKeysWords = W * kRowXposeWords + 4u + RowItems<EM, W, TMAX>::kWords + kMaxFanout + 1u;

template <int EM, int W, uint32_t TMAX, int MINW>
__global__ __launch_bounds__(W * 64, MINW) void k_merge_keys(Phase ph, Bufs b, RoundArgs ra,
                                                             const uint32_t* __restrict__ table, uint32_t flip) {
    using Items = RowItems<EM, W, TMAX>;
    const uint64_t L = ra.L;
    const uint32_t K = ra.K, Tout = ra.Tout;
    extern __shared__ __align__(16) uint32_t smem[];
    // split probes read up to 496 bytes before or after the keys
    static_assert(W * kRowXposeWords * 4u >= 496u && Items::kWords * 4u >= 496u, "LDS around the keys");
    uint32_t* X = smem + W * kRowXposeWords;
    uint32_t* sent = X + Tout + 4u * K;
    uint32_t* items = sent + 4u;
    uint32_t* sbeg = items + Items::kWords;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // wave-uniform
    uint32_t* wscr = smem + (uint32_t)wave * kRowXposeWords;
    const uint64_t t = blockIdx.x;
    const TileRef tr = tile_ref(ph, b, t);
    const uint32_t flip_out = tr.final_pass ? flip : 0u;
    const uint32_t grp = tr.local / (uint32_t)ra.tpg;
    const uint64_t i = tr.local - (uint64_t)grp * ra.tpg;
    const uint64_t span = (uint64_t)K * L;
    const uint64_t gb = (uint64_t)grp * span;
    const uint64_t glen = min(span, tr.n - gb);
    const uint32_t Kg = (uint32_t)((glen + L - 1) / L);
    const uint64_t obeg = i * (uint64_t)Tout;
    const uint32_t cnt = (uint32_t)min<uint64_t>(Tout, glen - obeg);
    const uint64_t obase = gb + obeg;

    if (Kg == 1) {   // a lone run: its tile is already in order
        for (uint32_t j = threadIdx.x; j < cnt; j += W * 64u)
            gptr(tr.dst_k)[obase + j] = gptr(tr.src_k)[obase + j] ^ flip_out;
        return;
    }
    // Every wave reads the tile's split indices (lane k < Kg: run k) and lays
    // the pieces out in registers, so its loads go out at once.
    uint32_t s = 0, e = 0;
    if ((uint32_t)lane < Kg) {
        const uint32_t k = (uint32_t)lane;
        const uint32_t nk = (uint32_t)min(L, glen - (uint64_t)k * L);
        // the clamps only guard memory safety; exact splits never trigger them
        s = i == 0 ? 0u : min(table[t * K + k], nk);
        e = (obeg + Tout >= glen) ? nk : min(max(table[(t + 1) * K + k], s), nk);
    }
    const PieceLayout pc = piece_layout(s, e, Kg, cnt, lane);
    const LoadSteps st = load_steps<8>(pc, s, Kg, L, lane);
    static_assert(TMAX / 256u + kMaxFanout < 64u, "a step per lane, and one lane without");
    cgu32* gk = gptr(tr.src_k) + gb;
    // A step reads 256 keys from its first on: a group of two runs or more holds
    // more than that, and the steps of its last ones come after the others, key
    // by key.  Steps past the last one read the group's first keys and store
    // nothing; lane 63 has none (above).
    const uint32_t gend = (uint32_t)glen - 256u;
    const bool late = (uint32_t)lane < st.total && st.src > gend;
    const uint32_t src = (uint32_t)lane < st.total ? min(st.src, gend) : 0u;
    const int len = (uint32_t)lane < st.total && !late ? (int)st.cnt : 0;
    constexpr uint32_t U = W == 8 ? 5 : 3;   // steps a wave has in flight
    for (uint32_t e0 = (uint32_t)wave; e0 < st.total; e0 += U * W) {
        u32x4a4 v[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const int x = (int)min(e0 + u * W, 63u);
            const uint32_t from = (uint32_t)__builtin_amdgcn_readlane((int)src, x);
            v[u] = *reinterpret_cast<cgu32x4a4*>(gk + from + 4u * (uint32_t)lane);
        }
        if (e0 == 0u) {   // wave 0 plans the levels while its first loads are in flight
            if ((uint32_t)lane < Kg) sbeg[lane] = pc.sb;
            const uint32_t end =
                (uint32_t)__builtin_amdgcn_readlane((int)(pc.sb + ((pc.len + 3u) & ~3u)), (int)(Kg - 1u));
            if (lane == 0) sbeg[Kg] = end;
            if (lane < 4) sent[lane] = kSentKey;
            lds_wave_sync();
            Items::build(items, sbeg, Kg, lane);
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const int x = (int)min(e0 + u * W, 63u);
            const int left = __builtin_amdgcn_readlane(len, x) - 4 * lane;
            const uint32_t dst = (uint32_t)__builtin_amdgcn_readlane((int)st.dst, x) + 4u * (uint32_t)lane;
            if (left > 0) {   // slots past the piece hold the largest key
                u32x4 k = v[u];
                k.y = left < 2 ? kSentKey : k.y;
                k.z = left < 3 ? kSentKey : k.z;
                k.w = left < 4 ? kSentKey : k.w;
                *reinterpret_cast<u32x4*>(X + dst) = k;
            }
        }
    }
    for (uint64_t todo = __ballot(late); todo; todo &= todo - 1u) {
        const int x = __builtin_ctzll(todo);
        const uint32_t from = (uint32_t)__builtin_amdgcn_readlane((int)st.src, x);
        const uint32_t dst = (uint32_t)__builtin_amdgcn_readlane((int)st.dst, x);
        const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)st.cnt, x);
        for (uint32_t j = threadIdx.x; j < ((n + 3u) & ~3u); j += W * 64u) X[dst + j] = j < n ? gk[from + j] : kSentKey;
    }
    lds_barrier();

    uint32_t nlev = 0;
    while ((1u << nlev) < Kg) ++nlev;
    const bool empty = __popcll(__ballot(pc.len != 0u)) < 1 << nlev;   // some pairs may have one run only
    uint32_t m[EM];
    RowOut o;
    for (uint32_t lvl = 0;;) {
        row_merge_level<EM, Items>(X, items, lvl, sent, wscr, wave, lane, empty && lvl + 1u < nlev, m, o);
        if (++lvl == nlev) break;
        row_put_lds(X, o, m, lane);
        lds_barrier();
    }
    gu32* g = gptr(tr.dst_k) + obase;
    row_put(o, m, lane, [&](int c, int step, uint32_t k0, uint32_t k1, uint32_t k2, uint32_t k3) {
        const u32x4 v{k0 ^ flip_out, k1 ^ flip_out, k2 ^ flip_out, k3 ^ flip_out};
        const uint32_t at = 4u * (uint32_t)(c + step);
        if (at + 4u <= cnt) {
            *reinterpret_cast<gu32x4a4*>(g + at) = v;
        } else {
#pragma unroll
            for (uint32_t j = 0; j < 4u; ++j)
                if (at + j < cnt) g[at + j] = v[j];
        }
    });
}

static hipError_t allow_lds(const void* f, size_t bytes) {
    if (bytes <= 64u << 10) return hipSuccess;   // what a launch may have without asking
    return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// TMAX: the largest merge tile of the shape.
template <int EM, int W, uint32_t TMAX, int MINW>
static hipError_t launch_variant(const Phase& ph, const Bufs& b, const RoundArgs& ra, const uint32_t* table,
                                 uint32_t flip, hipStream_t s) {
    if (ra.Tout > TMAX) return hipErrorInvalidValue;
    const size_t lds = (kMergeKeysWords<EM, W, TMAX> + ra.Tout + 4u * ra.K) * sizeof(uint32_t);
    hipError_t e = allow_lds((const void*)k_merge_keys<EM, W, TMAX, MINW>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_merge_keys<EM, W, TMAX, MINW>), dim3((unsigned)ph.tiles), dim3(W * 64), lds, s, ph, b, ra,
                       table, flip);
    return hipGetLastError();
}

hipError_t launch_merge_keys(const Phase& ph, const Bufs& b, const RoundArgs& ra, const uint32_t* table,
                             uint32_t flip, int variant, hipStream_t s) {
    if (ra.Tout > kToutKeys || ra.K > kMaxFanout || ra.Tout % 4 || ra.L % 4 || ra.L < 256)
        return hipErrorInvalidValue;
    if (ph.tiles == 0) return hipSuccess;
    if (variant == 4) return launch_merge_heap(ph, b, ra, table, flip, s);
    // a pass of rows holds any pair: eight waves of 256-key blocks up to
    // 7680-key tiles, of 128-key ones up to 3584, sixteen up to 7424 (a launch has
    // less than 2^32 threads: 2^32 - 1 keys in 1024-key tiles take eight waves)
    if (variant == 1 && ra.Tout <= 7424 && ph.tiles < 1u << 22)
        return launch_variant<8, 16, 7424, 8>(ph, b, ra, table, flip, s);
    if (variant == 2 && ra.Tout <= 3584) return launch_variant<8, 8, 3584, 8>(ph, b, ra, table, flip, s);
    if (ra.Tout <= 7680) return launch_variant<16, 8, 7680, 8>(ph, b, ra, table, flip, s);
    return launch_variant<16, 16, kToutKeys, 8>(ph, b, ra, table, flip, s);
}

}  // namespace mms
