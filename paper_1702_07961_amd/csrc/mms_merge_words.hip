// K-way merge rounds of the sorts whose elements are more than a 32-bit key
// (§4.2, values moving with their keys): stable (32-bit key, value) pairs.
// One workgroup per output tile.
//
// A tile's input is the K pieces of its group's runs bounded by the split
// indices of its first and last output (§4.1).  The pieces are laid out at
// 4-aligned LDS slots and become 64-bit words (key, slot) as they are loaded;
// the merge tree runs on the words, in place, in row blocks
// (mms_word_merge.h).  After the last level's reads the values take the words'
// place in LDS, and each is gathered by its word's tag as the keys are stored.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mms_device.h"
#include "mms_device_kt.h"
#include "mms_internal.h"
#include "mms_tile_plan.h"
#include "mms_word_merge.h"

namespace mms {

namespace {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// two elements at an address aligned to one
typedef uint32_t u32x2a4 __attribute__((ext_vector_type(2), aligned(4)));
typedef const __attribute__((address_space(1))) u32x2a4 cgu32x2a4;
typedef __attribute__((address_space(1))) u32x2 gu32x2;

// Pieces are loaded in steps of 128 elements, two per lane.  Step e of the
// tile sits in lane e of every wave: where its elements come from (in the
// group), its first LDS slot and its length.
struct LoadSteps {
    uint32_t src, dst, cnt, total;
};
__device__ __forceinline__ LoadSteps load_steps(const PieceLayout& pc, uint32_t s, uint32_t Kg, uint64_t L, int lane) {
    const uint32_t own = (pc.len + 127u) >> 7;   // lanes k < Kg hold piece k, the others none
    const uint32_t before = excl_scan16(own);
    uint32_t k = 0;
    for (uint32_t j = 0; j + 1u < Kg; ++j)   // pieces whose steps end at or before this lane's
        k += (uint32_t)__builtin_amdgcn_readlane((int)(before + own), (int)j) <= (uint32_t)lane ? 1u : 0u;
    const uint32_t from = (uint32_t)((uint64_t)(uint32_t)lane * L) + s;   // lane k: piece k's first element
    auto of = [&](uint32_t x) { return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(k << 2), (int)x); };
    const uint32_t at = ((uint32_t)lane - of(before)) << 7;
    LoadSteps r;
    r.src = of(from) + at;
    r.dst = of(pc.sb) + at;
    r.cnt = min(of(pc.len) - at, 128u);   // meaningful below total only
    r.total = (uint32_t)__builtin_amdgcn_readlane((int)(before + own), (int)(Kg - 1u));
    return r;
}

}  // namespace

// Bound by VALU issue (74 % of the launch's cycles; LDS half of them).  LDS
// holds one 8-byte word per element and nothing else that grows with the tile,
// so four workgroups of four waves share a compute unit.  2^27 pairs, K = 16:
// 0.81 ms per launch on average, where 512-pair blocks of a wave (two level
// buffers of keys and tags, the values in LDS throughout, two workgroups of
// eight waves) took 1.06.  With the values in LDS throughout and all lane
// distances by DPP, three workgroups fit: 0.92.
template <int EM, uint32_t TOUT, int W>
__global__ __launch_bounds__(W * 64, EM == 16 ? 4 : 6) void k_merge_pairs(Phase ph, Bufs b, RoundArgs ra,
                                                           const uint32_t* __restrict__ table, uint32_t flip) {
    using Items = WordItems<EM, TOUT, W>;
    constexpr uint32_t CAP = Items::kCap;
    const uint32_t Tout = ra.Tout, K = ra.K;
    const uint64_t L = ra.L;
    // split probes read up to 504 bytes before or after the words
    __shared__ struct __align__(16) {
        uint32_t scr[W * kWordXposeWords];
        double X[CAP];
        double sent[2];
        uint32_t items[Items::kWords];
        uint32_t sbeg[kMaxFanout + 1u];
    } sm;
    static_assert(Items::kWords * 4u >= 504u && W * kWordXposeWords * 4u >= 504u, "LDS around the words");
    double* X = sm.X;
    double* sent = sm.sent;
    uint32_t* items = sm.items;
    uint32_t* sbeg = sm.sbeg;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // wave-uniform
    uint32_t* wscr = sm.scr + (uint32_t)wave * kWordXposeWords;
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
        for (uint32_t j = threadIdx.x; j < cnt; j += blockDim.x) {
            gptr(tr.dst_k)[obase + j] = gptr(tr.src_k)[obase + j] ^ flip_out;
            gptr(tr.dst_v)[obase + j] = gptr(tr.src_v)[obase + j];
        }
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
    const LoadSteps st = load_steps(pc, s, Kg, L, lane);
    cgu32* gk = gptr(tr.src_k) + gb;
    const uint32_t glast = (uint32_t)glen - 2u;   // a group of two runs or more holds more than a base tile
    constexpr uint32_t U = 32 / W;                   // steps a wave has in flight
    for (uint32_t e0 = (uint32_t)wave; e0 < st.total; e0 += U * W) {
        u32x2 kv[U];
        uint32_t dst[U], left[U], back[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {   // steps past the last one load it again and store nothing
            const uint32_t x = min(e0 + u * W, st.total - 1u);
            const uint32_t src = (uint32_t)__builtin_amdgcn_readlane((int)st.src, (int)x);
            const uint32_t q = src + 2u * (uint32_t)lane;
            const uint32_t qc = min(q, glast);   // the group's last element is read one early
            back[u] = q - qc;
            kv[u] = *reinterpret_cast<cgu32x2a4*>(gk + qc);
            dst[u] = (uint32_t)__builtin_amdgcn_readlane((int)st.dst, (int)x) + 2u * (uint32_t)lane;
            left[u] = e0 + u * W < st.total ? (uint32_t)__builtin_amdgcn_readlane((int)st.cnt, (int)x) : 0u;
        }
        if (e0 == 0u) {   // wave 0 plans the levels while its first loads are in flight
            if ((uint32_t)lane < Kg) sbeg[lane] = pc.sb;
            const uint32_t end =
                (uint32_t)__builtin_amdgcn_readlane((int)(pc.sb + ((pc.len + 3u) & ~3u)), (int)(Kg - 1u));
            if (lane == 0) {
                sbeg[Kg] = end;
                sent[0] = sent[1] = kt_sentinel();
            }
            lds_wave_sync();
            Items::build(items, sbeg, Kg, lane);
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t l2 = 2u * (uint32_t)lane;
            if (l2 < ((left[u] + 3u) & ~3u)) {   // slots past the piece hold the sentinel
                const uint32_t k0 = back[u] ? kv[u].y : kv[u].x;
                const double w0 = l2 < left[u] ? kt_pack(k0, dst[u]) : kt_sentinel();
                const double w1 = l2 + 1u < left[u] ? kt_pack(kv[u].y, dst[u] + 1u) : kt_sentinel();
                *reinterpret_cast<d2*>(X + dst[u]) = d2{w0, w1};
            }
        }
    }
    lds_barrier();

    uint32_t nlev = 0;
    while ((1u << nlev) < Kg) ++nlev;
    double m[EM];
    WordRow o;
    for (uint32_t lvl = 0;;) {
        word_merge_level<EM, Items>(X, items, lvl, sent, wscr, wave, lane, m, o);
        if (++lvl == nlev) break;
        word_put_lds(X, o, m, lane);
        lds_barrier();
    }
    // the words are read: their slots take the values, which the outputs
    // gather by tag
    uint32_t* V = reinterpret_cast<uint32_t*>(X);
    for (uint32_t x = (uint32_t)wave; x < st.total; x += W) {
        const uint32_t src = (uint32_t)__builtin_amdgcn_readlane((int)st.src, (int)x);
        const uint32_t dst = (uint32_t)__builtin_amdgcn_readlane((int)st.dst, (int)x);
        const uint32_t len = (uint32_t)__builtin_amdgcn_readlane((int)st.cnt, (int)x);
        const uint32_t* from = tr.src_v + (gb + src);
        if ((uint32_t)lane < len) dma_dword(from, (uint32_t)lane, V + dst);
        if ((uint32_t)lane + 64u < len) dma_dword(from + 64, (uint32_t)lane, V + dst + 64u);
    }
    vm_drain();
    lds_barrier();
    gu32* ok = gptr(tr.dst_k) + obase;
    gu32* ov = gptr(tr.dst_v) + obase;
    const bool vec = (((uintptr_t)(tr.dst_k + obase) | (uintptr_t)(tr.dst_v + obase)) & 7u) == 0;
    word_row_put(o, m, lane, [&](uint32_t c, double a, double z) {
        const uint32_t at = 2u * c;
        if (vec && at + 2u <= cnt) {
            *reinterpret_cast<gu32x2*>(ok + at) = u32x2{kt_key(a) ^ flip_out, kt_key(z) ^ flip_out};
            *reinterpret_cast<gu32x2*>(ov + at) = u32x2{V[kt_tag(a)], V[kt_tag(z)]};
        } else {
            if (at < cnt) {
                ok[at] = kt_key(a) ^ flip_out;
                ov[at] = V[kt_tag(a)];
            }
            if (at + 1u < cnt) {
                ok[at + 1u] = kt_key(z) ^ flip_out;
                ov[at + 1u] = V[kt_tag(z)];
            }
        }
    });
}

hipError_t launch_merge_pairs(const Phase& ph, const Bufs& b, const RoundArgs& ra, const uint32_t* table,
                              uint32_t flip, hipStream_t s) {
    if (ph.tiles == 0) return hipSuccess;
    if (ra.Tout > kToutPairs || ra.Tout % 4 || ra.K > kMaxFanout) return hipErrorInvalidValue;
    // Up to as many tiles as are resident at once, one workgroup's latency is
    // what counts, and eight waves of 128-word blocks take half as long over a
    // level: 3.0e5 uniform pairs 79.1 us with the larger blocks and 71.1 with
    // these, 2e6 pairs (521 tiles) 136 and 130, 4e6 (1042) 210 and 204.  Past
    // that the larger blocks' fewer instructions win: 1e7 pairs 409 us and 416,
    // 1e8 3.97 ms and 4.19.
    if (ph.tiles <= 1024)
        hipLaunchKernelGGL((k_merge_pairs<8, kToutPairs, 8>), dim3((unsigned)ph.tiles), dim3(8 * 64), 0, s, ph, b, ra,
                           table, flip);
    else
        hipLaunchKernelGGL((k_merge_pairs<16, kToutPairs, 4>), dim3((unsigned)ph.tiles), dim3(4 * 64), 0, s, ph, b, ra,
                           table, flip);
    return hipGetLastError();
}

}  // namespace mms
