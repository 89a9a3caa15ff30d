// K-way merge rounds of the sorts whose elements are more than a 32-bit key
// (§4.2, §6.3): stable (32-bit key, value) pairs.
// One workgroup per output tile.
//
// A tile's input is the K pieces of its group's runs bounded by the split
// indices of its first and last output (§4.1).  The pieces are laid out at
// 4-aligned LDS slots and become 64-bit words (key, slot) as they are loaded;
// the merge tree runs on the words, in place, in row blocks
// (mms_word_merge.h).  After the last level's reads the values take the words'
// place in LDS, and each is gathered by its word's tag as the keys are stored.
//
// A word holds 64-bit keys alone whole where a tile's keys span less than 2^62.
// With their slot they do not fit, so the words of pairs (and of keys that span
// more) hold the leading 50 bits of the tile's range, and a tile that this did
// not put in order is set right afterwards (k_merge64 below).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "mms_device.h"
#include "mms_device64.h"
#include "mms_device_kt.h"
#include "mms_internal.h"
#include "mms_load_steps.h"
#include "mms_order64.h"
#include "mms_tile_plan.h"
#include "mms_word_merge.h"

namespace mms {

namespace {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) u32x2a4 cgu32x2a4;

}  // namespace

// Bound by VALU issue (74 % of the launch's cycles; LDS half of them).  LDS
// holds one 8-byte word per element and nothing else that grows with the tile,
// so four workgroups of four waves share a compute unit.  2^27 pairs, K = 16:
// 0.72 ms per launch on average (0.81 with items planned pair by pair, branching
// loads and 8-byte stores), where 512-pair blocks of a wave (two level buffers of
// keys and tags, the values in LDS throughout, two workgroups of eight waves) took
// 1.06.  With the values in LDS throughout and all lane
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
    const LoadSteps st = load_steps<7>(pc, s, Kg, L, lane);
    static_assert(TOUT / 128u + kMaxFanout < 64u, "a step per lane, and one lane without");
    cgu32* gk = gptr(tr.src_k) + gb;
    // A step reads 128 keys from its first on: a group of two runs or more holds
    // more than that, and the steps of its last ones come after the others, key
    // by key.  Steps past the last one read the group's first keys and store
    // nothing; lane 63 has none (above).
    const uint32_t gend = (uint32_t)glen - 128u;
    const bool late = (uint32_t)lane < st.total && st.src > gend;
    const uint32_t src = (uint32_t)lane < st.total ? min(st.src, gend) : 0u;
    const int len = (uint32_t)lane < st.total && !late ? (int)st.cnt : 0;
    constexpr uint32_t U = 40 / W;                   // steps a wave has in flight
    for (uint32_t e0 = (uint32_t)wave; e0 < st.total; e0 += U * W) {
        u32x2 kv[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const int x = (int)min(e0 + u * W, 63u);
            const uint32_t from = (uint32_t)__builtin_amdgcn_readlane((int)src, x);
            kv[u] = *reinterpret_cast<cgu32x2a4*>(gk + from + 2u * (uint32_t)lane);
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
            const int x = (int)min(e0 + u * W, 63u);
            const int n = __builtin_amdgcn_readlane(len, x), left = n - 2 * lane;
            const uint32_t dst = (uint32_t)__builtin_amdgcn_readlane((int)st.dst, x) + 2u * (uint32_t)lane;
            if (2 * lane < ((n + 3) & ~3)) {   // slots past the piece hold the sentinel
                const double w0 = left > 0 ? kt_pack(kv[u].x, dst) : kt_sentinel();
                const double w1 = left > 1 ? kt_pack(kv[u].y, dst + 1u) : kt_sentinel();
                *reinterpret_cast<d2*>(X + dst) = d2{w0, w1};
            }
        }
    }
    for (uint64_t todo = __ballot(late); todo; todo &= todo - 1u) {
        const int x = __builtin_ctzll(todo);
        const uint32_t from = (uint32_t)__builtin_amdgcn_readlane((int)st.src, x);
        const uint32_t dst = (uint32_t)__builtin_amdgcn_readlane((int)st.dst, x);
        const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)st.cnt, x);
        for (uint32_t j = threadIdx.x; j < ((n + 3u) & ~3u); j += W * 64u)
            X[dst + j] = j < n ? kt_pack(gk[from + j], dst + j) : kt_sentinel();
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
    word_row_put(o, m, lane, [&](int c, int step, double a, double z) {
        const uint32_t at = 2u * (uint32_t)(c + step);
        if (at + 2u <= cnt) {
            *reinterpret_cast<gu32x2a4*>(ok + at) = u32x2{kt_key(a) ^ flip_out, kt_key(z) ^ flip_out};
            *reinterpret_cast<gu32x2a4*>(ov + at) = u32x2{V[kt_tag(a)], V[kt_tag(z)]};
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

// ===========================================================================
// 64-bit keys, alone or with 64-bit values.
//
// Keys alone need no slots: where a tile spans less than 2^62 its words are the
// keys, and they are stored from the words.  Otherwise the words hold as much of
// the keys as fits with a slot (mms_order64.h); such words are unique and each
// piece's are in order, so the merge is exact in the order of the words.  The
// keys then come back into the words' place, to be checked and gathered.  A tile
// that is not in order merges its second words: a piece's are in order too, so
// its levels and items are the same.
// ===========================================================================
typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
typedef uint64_t u64x2a8 __attribute__((ext_vector_type(2), aligned(8)));
typedef const __attribute__((address_space(1))) u64x2a8 cgu64x2a8;
typedef __attribute__((address_space(1))) u64x2a8 gu64x2a8;

// Load the tile's elements (base: the group's first), each wave's share of the
// steps, up to U in flight: put(first slot of the lane's two, how many of the
// step's elements are left from there, the elements).  Lanes of a step's last
// four slots are called with none left.
template <uint32_t U, int W, class Mid, class Put>
__device__ __forceinline__ void load_u64(const uint64_t* base, uint32_t glast, const LoadSteps& st, int wave, int lane,
                                         const Mid& mid, const Put& put) {
    cgu64* g = gptr64(base);
    for (uint32_t e0 = (uint32_t)wave; e0 < st.total; e0 += U * W) {
        u64x2 v[U];
        uint32_t dst[U], back[U];
        int left[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {   // steps past the last one load it again and store nothing
            const uint32_t x = min(e0 + u * W, st.total - 1u);
            const uint32_t q = (uint32_t)__builtin_amdgcn_readlane((int)st.src, (int)x) + 2u * (uint32_t)lane;
            const uint32_t qc = min(q, glast);   // the group's last element is read one early
            back[u] = q - qc;
            v[u] = *reinterpret_cast<cgu64x2a8*>(g + qc);
            dst[u] = (uint32_t)__builtin_amdgcn_readlane((int)st.dst, (int)x) + 2u * (uint32_t)lane;
            const int n = e0 + u * W < st.total ? __builtin_amdgcn_readlane((int)st.cnt, (int)x) : 0;
            left[u] = 2 * lane < ((n + 3) & ~3) ? n - 2 * lane : -4;
        }
        mid(e0);
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
            if (left[u] > -4) put(dst[u], left[u], back[u] ? v[u].y : v[u].x, v[u].y);
    }
}

// Bound by VALU issue like the merge above.  Launch average of a sort, against
// blocks of 64-bit keys in their own order (a compare and four selects per
// compare-exchange): 10^8 keys 943 -> 567 us; 33,554,467 pairs 674 -> 277 us.
template <int EM, uint32_t TOUT, int W, bool PAIRS>
__global__ __launch_bounds__(W * 64, EM == 16 ? 4 : 6) void k_merge64(Phase64 ph, Bufs64 b, RoundArgs ra,
                                                                      const uint32_t* __restrict__ table,
                                                                      uint64_t flip) {
    using Items = WordItems<EM, TOUT, W>;
    constexpr uint32_t CAP = Items::kCap;
    constexpr uint32_t NT = W * 64u;
    static_assert(CAP < 1u << kSlotBits, "slots");
    const uint32_t Tout = ra.Tout, K = ra.K;
    const uint64_t L = ra.L;
    // split probes read up to 504 bytes before or after the words
    __shared__ struct __align__(16) {
        uint32_t scr[W * kWordXposeWords];
        double X[CAP];
        double sent[2];
        uint32_t items[Items::kWords];
        uint32_t sbeg[kMaxFanout + 1u];
        uint32_t send[kMaxFanout];
        Order64<W> order;
        uint32_t tags[CAP / 2u];   // the sorted slots, 16 bits each
    } sm;
    static_assert(Items::kWords * 4u >= 504u && W * kWordXposeWords * 4u >= 504u, "LDS around the words");
    double* X = sm.X;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // wave-uniform
    const uint32_t tid = threadIdx.x;
    uint32_t* wscr = sm.scr + (uint32_t)wave * kWordXposeWords;
    const uint64_t t = blockIdx.x;
    const uint64_t* src_k = ph.dst_out ? b.ws_k : b.out_k;
    const uint64_t* src_v = ph.dst_out ? b.ws_v : b.out_v;
    uint64_t* dst_k = ph.dst_out ? b.out_k : b.ws_k;
    uint64_t* dst_v = ph.dst_out ? b.out_v : b.ws_v;
    const uint64_t flip_out = ph.final_pass ? flip : 0ull;
    const uint32_t grp = (uint32_t)t / (uint32_t)ra.tpg;
    const uint64_t i = t - (uint64_t)grp * ra.tpg;
    const uint64_t span = (uint64_t)K * L;
    const uint64_t gb = (uint64_t)grp * span;
    const uint64_t glen = min(span, ph.n - gb);
    const uint32_t Kg = (uint32_t)((glen + L - 1) / L);
    const uint64_t obeg = i * (uint64_t)Tout;
    const uint32_t cnt = (uint32_t)min<uint64_t>(Tout, glen - obeg);
    const uint64_t obase = gb + obeg;

    if (Kg == 1) {   // a lone run: its tile is already in order
        for (uint32_t j = tid; j < cnt; j += NT) {
            gptr64(dst_k)[obase + j] = gptr64(src_k)[obase + j] ^ flip_out;
            if constexpr (PAIRS) gptr64(dst_v)[obase + j] = gptr64(src_v)[obase + j];
        }
        return;
    }
    uint32_t s = 0, e = 0;
    if ((uint32_t)lane < Kg) {
        const uint32_t k = (uint32_t)lane;
        const uint32_t nk = (uint32_t)min(L, glen - (uint64_t)k * L);
        // the clamps only guard memory safety; exact splits never trigger them
        s = i == 0 ? 0u : min(table[t * K + k], nk);
        e = (obeg + Tout >= glen) ? nk : min(max(table[(t + 1) * K + k], s), nk);
    }
    const PieceLayout pc = piece_layout(s, e, Kg, cnt, lane);
    const LoadSteps st = load_steps<7>(pc, s, Kg, L, lane);
    static_assert(TOUT / 128u + kMaxFanout <= 64u, "a step per lane");
    uint64_t kmin = ~0ull, kmax = 0;
    if (pc.len) {   // lanes of non-empty pieces
        cgu64* p = gptr64(src_k) + (gb + (uint64_t)(uint32_t)lane * L + s);
        kmin = p[0];
        kmax = p[pc.len - 1u];
    }
    const uint32_t glast = (uint32_t)glen - 2u;   // a group of two runs or more holds more than a base tile
    uint32_t shift = 0;
    // Keys alone that span less than 2^62: the words are the keys.  With slots, keys
    // of few ids and a small counter below them shared words in every round but the
    // last and were merged twice: 2*10^7 such keys (three to an id) 1208 -> 788 us,
    // 10^8 4979 -> 3562; uniform keys, checked and gathered then, 784 -> 724 and
    // 3696 -> 3481.
    bool direct = false;
    constexpr uint32_t U = 32 / W;                // steps a wave has in flight
    // Every wave takes the tile's smallest and largest key, whether it has a load
    // step or not (the last tile of a group may have fewer than waves): the
    // barriers further down stand in branches on shift, which all waves of the
    // workgroup must take alike.
    auto bounds = [&] {
        // row 0 holds the pieces
        kmax = lane_u64(row_extreme<true>(kmax), 0);
        kmin = lane_u64(row_extreme<false>(kmin), 0);
        shift = prefix_shift(kmax - kmin);
        direct = !PAIRS && (kmax - kmin) >> kKeyBits == 0u;
    };
    if ((uint32_t)wave >= st.total) bounds();
    load_u64<U, W>(
        src_k + gb, glast, st, wave, lane,
        [&](uint32_t e0) {
            if (e0 == (uint32_t)wave) bounds();
            if (e0 == 0u) {   // wave 0 plans the levels while its first loads are in flight
                if ((uint32_t)lane < Kg) {
                    sm.sbeg[lane] = pc.sb;
                    sm.send[lane] = pc.sb + pc.len;
                }
                const uint32_t end =
                    (uint32_t)__builtin_amdgcn_readlane((int)(pc.sb + ((pc.len + 3u) & ~3u)), (int)(Kg - 1u));
                if (lane == 0) {
                    sm.sbeg[Kg] = end;
                    sm.sent[0] = sm.sent[1] = kt_sentinel();
                    sm.order.bad = 0u;
                }
                lds_wave_sync();
                Items::build(sm.items, sm.sbeg, Kg, lane);
            }
        },
        [&](uint32_t slot, int left, uint64_t k0, uint64_t k1) {
            double w0, w1;
            if (direct) {
                w0 = left > 0 ? key_word(k0 - kmin) : kt_sentinel();
                w1 = left > 1 ? key_word(k1 - kmin) : kt_sentinel();
            } else {
                w0 = left > 0 ? order_word((k0 - kmin) >> shift, slot) : kt_sentinel();
                w1 = left > 1 ? order_word((k1 - kmin) >> shift, slot + 1u) : kt_sentinel();
            }
            *reinterpret_cast<d2*>(X + slot) = d2{w0, w1};
        });
    lds_barrier();

    uint32_t nlev = 0;
    while ((1u << nlev) < Kg) ++nlev;
    uint64_t* E = reinterpret_cast<uint64_t*>(X);
    auto store_lds = [&](uint32_t slot, int left, uint64_t a, uint64_t z) {
        if (left > 0) *reinterpret_cast<u64x2*>(E + slot) = u64x2{a, z};
    };
    for (bool exact = false;;) {
        double m[EM];
        WordRow o;
        for (uint32_t lvl = 0;;) {
            word_merge_level<EM, Items>(X, sm.items, lvl, sm.sent, wscr, wave, lane, m, o);
            if (++lvl == nlev) break;
            word_put_lds(X, o, m, lane);
            lds_barrier();
        }
        // left by `break`, as a return here moves spills into the levels (10^8 keys
        // 3759 -> 4190 us)
        if (direct) {
            gu64* g = gptr64(dst_k) + obase;
            word_row_put(o, m, lane, [&](int c, int step, double a, double z) {
                const uint32_t at = 2u * (uint32_t)(c + step);
                const uint64_t ka = (word_key(a) + kmin) ^ flip_out, kz = (word_key(z) + kmin) ^ flip_out;
                if (at + 2u <= cnt) *reinterpret_cast<gu64x2a8*>(g + at) = u64x2{ka, kz};
                else if (at < cnt) g[at] = ka;
            });
            break;
        }
        // the words are read: the keys take their place, by slot
        word_row_put(o, m, lane, [&](int c, int step, double a, double z) {
            (sm.tags + c)[step] = word_slot(a) | word_slot(z) << 16;
        });
        load_u64<U, W>(src_k + gb, glast, st, wave, lane, [](uint32_t) {}, store_lds);
        lds_barrier();
        if (exact || (PAIRS && shift == 0u) || sm.order.ordered(E, sm.tags, cnt, tid)) break;
        exact = true;
        sm.order.template second_words<(TOUT + NT - 1u) / NT>(E, sm.tags, cnt, kmin, shift, tid);
        if (tid < Kg)   // the slots past each piece hold the sentinel again
            for (uint32_t x = sm.send[tid]; x & 3u; ++x) X[x] = kt_sentinel();
        lds_barrier();
    }
    if (!direct) store_by_tags<NT>(dst_k + obase, E, sm.tags, cnt, flip_out, tid);
    if constexpr (PAIRS) {   // the values in the keys' place
        lds_barrier();
        load_u64<U, W>(src_v + gb, glast, st, wave, lane, [](uint32_t) {}, store_lds);
        lds_barrier();
        store_by_tags<NT>(dst_v + obase, E, sm.tags, cnt, 0ull, tid);
    }
}

hipError_t launch_merge_pairs(const Phase& ph, const Bufs& b, const RoundArgs& ra, const uint32_t* table,
                              uint32_t flip, hipStream_t s) {
    if (ph.tiles == 0) return hipSuccess;
    if (ra.Tout > kToutPairs || ra.Tout % 4 || ra.K > kMaxFanout || ra.L < 128) return hipErrorInvalidValue;
    // While a launch's tiles are resident at once, one workgroup's latency is what
    // counts, and eight waves of 128-word blocks take half as long over a level;
    // three such workgroups fit a compute unit (768 tiles at once), four of the
    // larger blocks (1024).  Sorts with these and with the larger blocks: 300 tiles
    // 102 and 108 us, 640 134 and 140; 768 147 and 144, 960 161 and 153 (a second
    // wave of workgroups here, one there); 1024 168 and 173, 1300 198 and 205;
    // 2048 the same.  Past that the larger blocks' fewer instructions win: 2605
    // tiles 332 and 327, 28000 3540 and 3339.  The line lies at the larger blocks'
    // residency.
    if (ph.tiles <= 1024)
        hipLaunchKernelGGL((k_merge_pairs<8, kToutPairs, 8>), dim3((unsigned)ph.tiles), dim3(8 * 64), 0, s, ph, b, ra,
                           table, flip);
    else
        hipLaunchKernelGGL((k_merge_pairs<16, kToutPairs, 4>), dim3((unsigned)ph.tiles), dim3(4 * 64), 0, s, ph, b, ra,
                           table, flip);
    return hipGetLastError();
}

template <bool PAIRS>
static hipError_t launch64(const Phase64& ph, const Bufs64& b, const RoundArgs& ra, const uint32_t* table,
                           uint64_t flip, hipStream_t s) {
    // as for the 32-bit pairs (the same workgroups fit): keys 300 tiles 92 and 98
    // us, 960 158 and 157, 1300 196 and 199, 5000 635 and 613, 28000 3490 and 3320;
    // pairs 99 and 108, 190 and 181, 234 and 244, 829 and 823, 4409 and 4265
    if (ph.tiles <= 1024)
        hipLaunchKernelGGL((k_merge64<8, kTout64, 8, PAIRS>), dim3((unsigned)ph.tiles), dim3(8 * 64), 0, s, ph, b, ra,
                           table, flip);
    else
        hipLaunchKernelGGL((k_merge64<16, kTout64, 4, PAIRS>), dim3((unsigned)ph.tiles), dim3(4 * 64), 0, s, ph, b, ra,
                           table, flip);
    return hipGetLastError();
}

hipError_t launch_merge64(bool pairs, const Phase64& ph, const Bufs64& b, const RoundArgs& ra, const uint32_t* table,
                          uint64_t flip, hipStream_t s) {
    if (ph.tiles == 0) return hipSuccess;
    if (ra.Tout > kTout64 || ra.Tout % 4 || ra.K > kMaxFanout) return hipErrorInvalidValue;
    return pairs ? launch64<true>(ph, b, ra, table, flip, s) : launch64<false>(ph, b, ra, table, flip, s);
}

}  // namespace mms
