// gfx950 kernels of the 64-bit multiway mergesort (§6.3 also sorts 8-byte
// integers): 64-bit keys alone, or stable pairs of 64-bit keys and 64-bit
// values.  The method is the one of the 32-bit path:
//
//   tile_net64    base case (§4.3): each workgroup sorts a tile of words in
//                 registers
//   corank64      partition (§4.1): the exact split of each output tile
//
// The K-way merges (§4.2, §7) are in mms_merge_words.hip.  Words carry an
// element's slot in its tile, so every step is stable; the values never enter
// the networks and are gathered by slot when a tile is stored.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mms_corank.h"
#include "mms_device.h"
#include "mms_device64.h"
#include "mms_internal.h"
#include "mms_order64.h"
#include "mms_tile_net.h"

namespace mms {

// ===========================================================================
// Base case: the network of mms_tile_net.h on words that hold as much of the
// keys as fits (mms_order64.h).  A thread keeps its keys in registers: they go
// where the words were to be checked, and again if the tile is sorted twice.
// 10^8 keys 1244 -> 595 us against a network of 64-bit keys with an exchange for
// every lane and wave distance (8 per lane x 8 waves); 33,554,467 pairs 774 ->
// 243 us against one of keys and tags (2048-pair tiles).  A tile that is sorted
// twice takes longer than that network up to 10^5 elements or so (4000 keys 18.4
// us, 24.4 here; 10^6 131 and 109).
// ===========================================================================
template <int W, bool PAIRS>
__global__ __launch_bounds__(W * 64, 3) void k_tile_sort_net64(Phase64 ph, Bufs64 b, uint64_t flip) {
    constexpr uint32_t T = 1024u * W, NT = W * 64u;
    static_assert(T <= 1u << kSlotBits, "slots");
    __shared__ struct __align__(16) {
        double X[net_words<double>(T)];
        uint32_t tags[T / 2u];   // the sorted slots, 16 bits each
        uint64_t lo[W], hi[W], ones[W];
        Order64<W> order;
    } sm;
    const int lane = threadIdx.x & 63;
    const uint32_t ul = (uint32_t)lane, tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t base = (uint64_t)blockIdx.x * T;
    const uint32_t cnt = (uint32_t)min<uint64_t>(T, ph.n - base);
    const uint64_t flip_out = ph.final_pass ? flip : 0ull;
    typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
    typedef uint64_t u64x2a8 __attribute__((ext_vector_type(2), aligned(8)));
    typedef const __attribute__((address_space(1))) u64x2a8 cgu64x2a8;
    // Elements at + 128c and the next one are the thread's (c < 8).  The loads are
    // the same for all lanes: past the tile's end they bring in its last element,
    // which changes neither the bounds nor the bits below.  A wave past the end has
    // none.
    const uint32_t at = (uint32_t)wave * 1024u + 2u * ul;
    const bool some = (uint32_t)wave * 1024u < cnt;
    auto load = [&](const uint64_t* in, uint64_t (&r)[kNetRegs], uint64_t x) {
        if (cnt == 1u) {
#pragma unroll
            for (uint32_t e = 0; e < kNetRegs; ++e) r[e] = gptr64(in)[base] ^ x;
        } else if (some) {
#pragma unroll
            for (uint32_t c = 0; c < 8u; ++c) {
                const uint32_t j = at + 128u * c, q = min(j, cnt - 2u);
                const u64x2a8 v = *reinterpret_cast<cgu64x2a8*>(gptr64(in) + base + q);
                r[2 * c] = (q == j ? v.x : v.y) ^ x;
                r[2 * c + 1] = v.y ^ x;
            }
        }
    };
    uint64_t* E = reinterpret_cast<uint64_t*>(sm.X);
    auto put = [&](const uint64_t (&r)[kNetRegs]) {
#pragma unroll
        for (uint32_t c = 0; c < 8u; ++c) *reinterpret_cast<u64x2*>(E + at + 128u * c) = u64x2{r[2 * c], r[2 * c + 1]};
    };

    uint64_t key[kNetRegs] = {};
    load(b.in_k, key, flip);
    uint64_t kmin = ~0ull, kmax = 0, ones = 0;
    if (some) {
#pragma unroll
        for (uint32_t r = 0; r < kNetRegs; ++r) {
            kmin = min(kmin, key[r]);
            kmax = max(kmax, key[r]);
            ones |= key[r];
        }
        kmin = row_extreme<false>(kmin);
        kmax = row_extreme<true>(kmax);
        ones = row_reduce(ones, [](uint64_t a, uint64_t b) { return a | b; });
    }
    {
        const uint64_t lo = min(min(lane_u64(kmin, 0), lane_u64(kmin, 16)), min(lane_u64(kmin, 32), lane_u64(kmin, 48)));
        const uint64_t hi = max(max(lane_u64(kmax, 0), lane_u64(kmax, 16)), max(lane_u64(kmax, 32), lane_u64(kmax, 48)));
        const uint64_t any = lane_u64(ones, 0) | lane_u64(ones, 16) | lane_u64(ones, 32) | lane_u64(ones, 48);
        if (lane == 0) {
            sm.lo[wave] = lo;
            sm.hi[wave] = hi;
            sm.ones[wave] = any;
        }
        if (tid == 0) sm.order.bad = 0u;
    }
    lds_barrier();
    kmin = sm.lo[0];
    kmax = sm.hi[0];
    ones = sm.ones[0];
#pragma unroll
    for (int w = 1; w < W; ++w) {
        kmin = min(kmin, sm.lo[w]);
        kmax = max(kmax, sm.hi[w]);
        ones |= sm.ones[w];
    }
    kmin = lane_u64(kmin, 0);   // the same in every lane
    kmax = lane_u64(kmax, 0);
    const uint32_t shift = prefix_shift(kmax - kmin);
    bool exact = shift == 0u;   // the words hold the keys' whole order

    double m[kNetRegs];
    auto words = [&](const auto& order) {
#pragma unroll
        for (uint32_t r = 0; r < kNetRegs; ++r) {
            const uint32_t slot = at + 128u * (r >> 1) + (r & 1u);
            m[r] = slot < cnt ? order_word(order(key[r]), slot) : kt_sentinel();
        }
    };
    // Composite keys, an id in the high half and a counter in the low bits, fit
    // without the bits between: 4000 keys, three to an id, 25.5 -> 12.7 us
    // (which sorted nearly every such tile twice), 10^6 103 -> 89; uniform keys,
    // with the loads above, 14.5 -> 14.1 and 91.6 -> 90.4.
    KeyGap gap{};
    if (!exact) gap = key_gap(lane_u64(ones, 0), kmin, kmax, shift);
    if (gap.fits) {
        exact = true;
        words([&](uint64_t k) { return without_gap(k, gap); });
    } else {
        words([&](uint64_t k) { return (k - kmin) >> shift; });
    }
    for (;;) {
        net_sort<NetWord, W>(sm.X, m, cnt, lane, wave);
        uint32_t* t = sm.tags + (uint32_t)wave * 512u + ul * 8u;   // layout A: 16 positions in a row
#pragma unroll
        for (uint32_t r = 0; r < 8u; ++r) t[r] = word_slot(m[2 * r]) | word_slot(m[2 * r + 1]) << 16;
        lds_barrier();
        put(key);
        lds_barrier();
        if (exact || sm.order.ordered(E, sm.tags, cnt, tid)) break;
        exact = true;
        sm.order.template second_words<T / NT>(E, sm.tags, cnt, kmin, shift, tid);
        lds_barrier();
#pragma unroll
        for (uint32_t r = 0; r < kNetRegs; ++r) {
            const uint32_t slot = at + 128u * (r >> 1) + (r & 1u);
            m[r] = slot < cnt ? sm.X[slot] : kt_sentinel();
        }
        lds_barrier();
    }
    store_by_tags<NT>((ph.dst_out ? b.out_k : b.ws_k) + base, E, sm.tags, cnt, flip_out, tid);
    if constexpr (PAIRS) {
        load(b.in_v, key, 0ull);
        lds_barrier();
        put(key);
        lds_barrier();
        store_by_tags<NT>((ph.dst_out ? b.out_v : b.ws_v) + base, E, sm.tags, cnt, 0ull, tid);
    }
}

// ===========================================================================
// Partition (§4.1): one wave per output tile of a merge round, the split at
// the tile's first output.  The round reads the buffer it does not write.
// ===========================================================================
__global__ __launch_bounds__(256) void k_corank_tiles64(Phase64 ph, Bufs64 b, RoundArgs ra,
                                                        uint32_t* __restrict__ table) {
    __shared__ CorankLdsT<uint64_t> sh[4];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t t = (uint64_t)blockIdx.x * 4u + (uint64_t)wave;
    if (t >= ph.tiles) return;
    const uint64_t* src = ph.dst_out ? b.ws_k : b.out_k;
    const uint64_t grp = t / ra.tpg;
    const uint64_t i = t - grp * ra.tpg;
    const uint64_t span = (uint64_t)ra.K * ra.L;
    const uint64_t gb = grp * span;
    const uint64_t glen = min(span, ph.n - gb);
    const uint32_t Kg = (uint32_t)((glen + ra.L - 1) / ra.L);
    uint32_t c = 0;
    if (i > 0) c = corank_wave<uint64_t>(src, gb, glen, ra.L, Kg, (uint32_t)(i * ra.Tout), 0ull, lane, &sh[wave]);
    if ((uint32_t)lane < ra.K) table[t * ra.K + (uint64_t)lane] = c;
}

// ===========================================================================
// Launchers
// ===========================================================================
hipError_t launch_tile_sort64(bool pairs, const Phase64& ph, const Bufs64& b, uint64_t flip, hipStream_t s) {
    if (ph.tiles == 0) return hipSuccess;
    constexpr int W = kT64Waves;
    const dim3 grid((unsigned)ph.tiles), block(W * 64);
    if (pairs) hipLaunchKernelGGL((k_tile_sort_net64<W, true>), grid, block, 0, s, ph, b, flip);
    else hipLaunchKernelGGL((k_tile_sort_net64<W, false>), grid, block, 0, s, ph, b, flip);
    return hipGetLastError();
}

hipError_t launch_corank_tiles64(const Phase64& ph, const Bufs64& b, const RoundArgs& ra, uint32_t* table,
                                 hipStream_t s) {
    if (ph.tiles == 0) return hipSuccess;
    const uint64_t blocks = (ph.tiles + 3) / 4;
    hipLaunchKernelGGL(k_corank_tiles64, dim3((unsigned)blocks), dim3(256), 0, s, ph, b, ra, table);
    return hipGetLastError();
}

}  // namespace mms
