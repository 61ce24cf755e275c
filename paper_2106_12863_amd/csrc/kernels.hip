// libsinet kernels: per-session discrimination fused with the millisecond
// histogram, for gfx950.
//
// Method (Ando et al., arXiv 2106.12863):
//   * Algorithm 1: an address is inside a CIDR block when
//     bitmask(addr, Z) - bitmask(base, Z) == 0; applied to both endpoints of a
//     session against the whole table, it yields the label
//     in(src) | in(dst) << 1.
//   * Sections "Map" / "Reduce" / "Merge Scatter Pattern": every session maps
//     to key (label, floor((ts - t0) / width)) with value (1, bytes); values
//     merge by unsigned 64-bit addition, associative and commutative, so the
//     order of accumulation is free and the result is exact.
//
// GPU design (what differs from the paper's Thrust transform + pairwise
// reduction + CPU merge):
//   * stage 1 (k_stage1): each lane owns 4 consecutive sessions, read with
//     128-bit loads per column (two for the 64-bit byte column) one chunk
//     ahead; it classifies them against the table staged in LDS, writes the
//     4 labels as one 32-bit store, and counting-sorts the chunk by 1,024-bin
//     block into 4-byte records;
//   * stage 2 (k_stage2): persistent workgroups reduce one block's records in
//     LDS and write every bin of the block once; no zero-fill and no global
//     atomics on the hot path; sessions outside a chunk's block window take
//     a far pass with device-scope atomics, so any input order stays exact;
//   * lookups that walk global memory (trie, learned windows, binary search
//     with a global leaf) run as their own pass that stores the labels first;
//   * the batched form runs the same stages over many streams from device
//     work queues, captured in one graph.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string.h>

#include <algorithm>
#include <atomic>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "inout_index.h"
#include "local_shape.h"
#include "pass_common.h"
#include "sinet_device.h"
#include "sinet_internal.h"

namespace sinet {

enum KernelKind : uint32_t {
    KK_SCAN = SINET_LOOKUP_SCAN,
    KK_BSEARCH = SINET_LOOKUP_BSEARCH,
    KK_TRIE = SINET_LOOKUP_TRIE,
    KK_PLA = SINET_LOOKUP_LEARNED_PLA,
    KK_MLP = SINET_LOOKUP_LEARNED_MLP,
    KK_INOUT = kInoutKind,  // label-only lookups through the in/out index
    KK_UNION = kUnionKind,  // label-only lookups of a scan table: its union's boundaries
    KK_LABEL_IN = 100       // histogram of given labels
};
static_assert(KK_LABEL_IN == kLabelInKind && KK_INOUT == kInoutKind && KK_UNION == kUnionKind,
              "internal kinds");

constexpr int kXcds = 8;
constexpr int kMaxBlock = 1024;
constexpr int kStage2Block = 512;
constexpr int kSegMax = 256;               // segment descriptors of a block held in LDS
constexpr int kRecUnroll = 8;              // independent record loads per stage-2 lane
constexpr uint32_t kStage2Run = 16;         // consecutive stage-2 blocks per XCD turn (rows off a line)
constexpr uint32_t kSmallMax = 1u << 19;  // byte counts stored inline in a record
constexpr uint64_t kMaxPiece = 1ull << 31;  // sessions per partitioned pass (32-bit slots)

// ---------------------------------------------------------------------------
// searches
//
// A lane looks up several addresses at once (its four sessions' sources and
// destinations).  Every search below advances all of them in lockstep, one
// probe level at a time, so a lane keeps that many independent LDS or global
// loads in flight instead of waiting out one dependent chain per address.
// ---------------------------------------------------------------------------

// Per-workgroup LDS view of the table.  The pointers say that they address LDS:
// through generic pointers that are chosen at run time (a filter in LDS or in
// device memory, a view set inside a loop over streams) the compiler reads LDS
// with flat loads, which take both kinds of memory's paths and waits.
typedef const __attribute__((address_space(3))) uint32_t* lds_u32;
typedef const __attribute__((address_space(3))) float* lds_f32;
struct LdsView {
    lds_u32 io;      // in/out index, or the union's boundaries
    lds_u32 filter;  // 2-bit state of every /16 block (interval kinds)
    lds_u32 top;     // BSEARCH
    lds_u32 member;  // all interval kinds, when it is in LDS
    lds_u32 cb;      // SCAN
    lds_u32 mask;
    lds_u32 len;
    lds_u32 knot;    // PLA
    lds_f32 c;
    lds_f32 g;
    lds_u32 radix;   // PLA: first segment of each radix bucket (u16 pairs)
    lds_f32 w;       // MLP
    __attribute__((address_space(3))) uint32_t* queue;  // lookup pass of the interval kinds: this wave's search queue
};

// Membership bit of interval j.
__device__ __forceinline__ uint32_t member_bit(const DevTable& t, const LdsView& v, uint32_t j) {
    const uint32_t w = t.lds_member_words ? v.member[j >> 5] : *glob(t.member + (j >> 5));
    return (w >> (j & 31u)) & 1u;
}

// Entries of a wave's search queue: the searches of the 8 address slots (4
// sessions) of the wave's 64 lanes.
constexpr uint32_t kSearchQueue = 512;

// The window PLA's queue per wave: a ring of 128 addresses (fewer than 64 wait
// when a slot's up to 64 are added; the PLA's tables leave little LDS beside
// them).
constexpr uint32_t kPlaQueue = 128;

// Kinds whose lookup pass queues its searches: the binary searches, the trie,
// the MLP and the PLA.  The window PLA reads each queued window with a pair of
// lanes; the kinds whose search ends in a leaf of B in global memory (the
// LDS-sampled binary search, the MLP, a PLA with a wider bound) read each
// queued leaf with a pair of lanes, one round trip instead of a dependent
// binary search (read by quads, on the 1.6e9-session day: sampled binary search
// 18.9 -> 11.2 ms, MLP 23.2 -> 14.4 ms, 256-segment PLA 24.4 -> 13.2 ms; the
// same PLA queued with its leaf binary searches was slower than unqueued, 24.3
// -> 37.5 ms.  Pairs instead of quads, 2e8 addresses of clustered prefixes:
// sampled binary search 1.42 -> 1.31 ms, MLP 1.90 -> 1.83 ms; and without
// conditional loads, the filter's answer taken as it is: 1.22 and 1.70 ms).
__host__ __device__ constexpr bool queued_kind(uint32_t kind) {
    return kind == KK_BSEARCH || kind == KK_TRIE || kind == KK_MLP || kind == KK_PLA;
}

// Which queued searches a lookup instantiates (a template flag set): the
// window PLA's, the others' (binary searches, trie, MLP, wider PLA), or both.
constexpr int kQueueWindow = 1;
constexpr int kQueueSearch = 2;
constexpr int kQueueAll = kQueueWindow | kQueueSearch;

// Orders this wave's LDS accesses: the ones before complete before the ones
// after are issued (a wave's LDS requests are served in order; the clobber
// keeps the compiler from moving accesses across).
__device__ __forceinline__ void lds_wave_sync() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// For each q: the last arr[i] <= a[q] among arr[0..n), given arr[0] <= a[q].
template <int N>
__device__ __forceinline__ void upper_last_n(lds_u32 arr, uint32_t n, const uint32_t* a, uint32_t* lo) {
#pragma unroll
    for (int q = 0; q < N; ++q) lo[q] = 0;
    while (n > 1) {
        const uint32_t half = n >> 1;
#pragma unroll
        for (int q = 0; q < N; ++q) lo[q] = (arr[lo[q] + half] <= a[q]) ? lo[q] + half : lo[q];
        n -= half;
    }
}

__device__ __forceinline__ uint32_t radix_entry(lds_u32 radix, uint32_t i) {
    return (radix[i >> 1] >> ((i & 1) * 16)) & 0xFFFFu;
}

// Leaf phase shared by the binary search and the learned kinds: j[q] holds a
// leaf-block index (an index into the sampled boundaries); the leaf's
// 2^top_log2 boundaries (one or two cache lines, padded with 0xFFFFFFFF) are
// searched in global memory.
template <int N>
__device__ __forceinline__ void leaf_search(const DevTable& t, const uint32_t* a, uint32_t* j,
                                            uint32_t need) {
    if (t.top_log2 == 0) return;
#pragma unroll
    for (int q = 0; q < N; ++q) j[q] <<= t.top_log2;
    uint32_t n = 1u << t.top_log2;
    while (n > 1) {
        const uint32_t half = n >> 1;
        // (a plain pointer: with a global one the search of a whole day over B
        // took 56.4 ms instead of 55.0)
#pragma unroll
        for (int q = 0; q < N; ++q)
            if ((need >> q) & 1u) j[q] = (t.B[j[q] + half] <= a[q]) ? j[q] + half : j[q];
        n -= half;
    }
#pragma unroll
    for (int q = 0; q < N; ++q) j[q] = min(j[q], t.m - 1);
}

// Learned forms: the model's rounded prediction p is within max_err = e of
// the true interval j for every boundary key.  The leaf blocks that
// [p - e, p + e] can touch are searched in the LDS copy of the sampled
// boundaries (a window of uniform length, shifted inside the array) and the
// bracket top[b] <= a < top[b + 1] is confirmed, giving the leaf block b; the
// leaf is then searched as in the plain binary search.  A failed bracket (a
// wrong model or bound) falls back to the full search over the sample and is
// counted, so results stay exact.
template <int N>
__device__ __forceinline__ void learned_top_n(const DevTable& t, const LdsView& v,
                                              const uint32_t* a, const int* p, uint32_t* j,
                                              uint32_t need) {
    const uint32_t L = t.top_log2;
    const uint32_t nbl = min(((2 * t.max_err) >> L) + 2, t.n_top);
    uint32_t b[N], first[N];
    bool ok[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const int lo = max(p[q] - (int)t.max_err, 0);
        uint32_t b0 = (uint32_t)lo >> L;
        b0 = min(b0, t.n_top - nbl);
        first[q] = b0;
        b[q] = b0;
        ok[q] = v.top[b0] <= a[q];
    }
    uint32_t n = nbl;
    while (n > 1) {
        const uint32_t half = n >> 1;
#pragma unroll
        for (int q = 0; q < N; ++q) b[q] = (v.top[b[q] + half] <= a[q]) ? b[q] + half : b[q];
        n -= half;
    }
#pragma unroll
    for (int q = 0; q < N; ++q) {
        if (!((need >> q) & 1u)) continue;
        const uint32_t last = first[q] + nbl - 1;
        if (ok[q] && b[q] == last && last + 1 < t.n_top && v.top[last + 1] <= a[q]) ok[q] = false;
        if (!ok[q]) {
            atomicAdd(t.fallbacks, 1ull);
            b[q] = upper_last(v.top, t.n_top, a[q]);
        }
        j[q] = b[q];
    }
}

// The learned search: leaf block from the LDS sample, then the leaf.
template <int N>
__device__ __forceinline__ void learned_search_n(const DevTable& t, const LdsView& v,
                                                 const uint32_t* a, const int* p, uint32_t* j,
                                                 uint32_t need) {
    learned_top_n<N>(t, v, a, p, j, need);
    leaf_search<N>(t, a, j, need);
}

// PLA window search (max_err = e <= kPlaWindowErr): the interval of a lies
// within e of the rounded prediction p, so the 16 boundaries from
// s = (p - e) rounded down to a multiple of 4 hold it.  They are read with
// four aligned 16-byte loads, and B[s + 16] with them (two addresses'
// windows in flight at once), and j = s + (the number of them <= a) - 1.  A
// count of 0, or of 16 with B[s + 16] <= a, means the bound was wrong: the
// full search answers, counted.
template <int N>
__device__ __forceinline__ void window_search_n(const DevTable& t, const uint32_t* a, const int* p,
                                                uint32_t* j, uint32_t need) {
    constexpr int G = N < 2 ? N : 2;
    const int e = (int)t.max_err;
#pragma unroll
    for (int q0 = 0; q0 < N; q0 += G) {
        uint4 w[G][4];
        uint32_t s[G], nx[G];
#pragma unroll
        for (int q = 0; q < G; ++q) {
            s[q] = (uint32_t)max(p[q0 + q] - e, 0) & ~3u;
            if ((need >> (q0 + q)) & 1u) {
                const uint32_t* b4 = t.B + s[q];
#pragma unroll
                for (int v = 0; v < 4; ++v) w[q][v] = gload4(b4 + 4 * v);
                nx[q] = *glob(t.B + s[q] + 16u);  // for the bracket check (in the padding at worst)
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v) w[q][v] = make_uint4(0u, 0u, 0u, 0u);
                nx[q] = 0xFFFFFFFFu;
            }
        }
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int qq = q0 + q;
            if (!((need >> qq) & 1u)) continue;
            const uint32_t x = a[qq];
            uint32_t c = 0;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                c += (uint32_t)(w[q][v].x <= x) + (uint32_t)(w[q][v].y <= x) +
                     (uint32_t)(w[q][v].z <= x) + (uint32_t)(w[q][v].w <= x);
            bool ok = c >= 1u;
            if (c == 16u && s[q] + 16u < t.m) ok = x < nx[q];
            uint32_t r = s[q] + c - 1u;
            if (!ok) {
                atomicAdd(t.fallbacks, 1ull);
                r = upper_last(glob(t.B), t.m, x);
            }
            j[qq] = min(r, t.m - 1);
        }
    }
}

// Lane index within the wave.
__device__ __forceinline__ uint32_t lane_id() {
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// Rank of this lane among the lanes set in m.
__device__ __forceinline__ uint32_t rank_in(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// x of lane src (every lane active).
__device__ __forceinline__ uint32_t from_lane(uint32_t src, uint32_t x) {
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(src << 2), (int)x);
}

// Sum over the two lanes of each pair, in both (DPP quad permutation [1,0,3,2];
// every lane active).
__device__ __forceinline__ uint32_t pair_sum(uint32_t x) {
    return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, false);
}

// One round of the window PLA's queue: the membership bits of the nr <= 64
// addresses at places head.. of the wave's ring, one bit per address in order.
// Lane s takes the address of place E(s) = 2 (s mod 32) + s / 32, finds its
// segment, evaluates the line and forms the window's first index; then, in two
// steps of 32 addresses, each pair of lanes takes one address (moved over with
// ds_bpermute), each lane loads and compares eight of the 16 boundaries, and
// the pair's counts are added with DPP.  One load instruction covers half of 32
// windows.  The lane at place k of a pair then finishes the pair's address of
// step k, which by the choice of E is the address whose place is that lane's
// own index: it checks the bracket (falling back to the full search, counted,
// as window_search_n does) and reads the interval's membership bit.  The
// boundary after a window is read only where all 16 are <= the address: read
// with the window for every address it took up to 64 cache lines per round
// (5e8 labels 3.47 -> 3.27 ms without).
// The pass is bound by VALU issue, and a step's moves, address arithmetic and
// sum cost more than a load: with pairs a round has two steps, with quads it
// had four (5e8 labels of the 1024-segment table, together with the LDS-typed
// pointers, 4.05 -> 3.74 ms).
__device__ __forceinline__ unsigned long long pla_round(const DevTable& t, const LdsView& v,
                                                        uint32_t head, uint32_t nr, uint32_t lane) {
    const int e = (int)t.max_err;
    const uint32_t place = ((lane & 31u) << 1) | (lane >> 5);
    // (a lane without an address searches address 0, in bounds like any other,
    // and its bit is dropped: no load is conditional)
    const uint32_t x = place < nr ? v.queue[(head + place) & (kPlaQueue - 1u)] : 0u;
    // radix bucket -> candidate segments -> last knot <= x -> line
    const uint32_t rb = x >> (32 - t.radix_bits);
    const uint32_t s0 = radix_entry(v.radix, rb), s1 = radix_entry(v.radix, rb + 1);
    const uint32_t sg = s0 + upper_last(v.knot + s0, s1 - s0 + 1, x);
    const int pp = clamp_pos(pla_eval(v.knot[sg], v.c[sg], v.g[sg], x), t.m);
    const uint32_t wb = (uint32_t)max(pp - e, 0) & ~3u;
    // every window load is issued before any is used
    const uint32_t me = lane & 1u;
    uint32_t xx[2], bb[2], c[2];
    uint4 w[2][2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const uint32_t src = 32u * k + (lane >> 1);
        xx[k] = from_lane(src, x);
        bb[k] = from_lane(src, wb);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        w[k][0] = gload4(t.B + bb[k] + 4u * me);
        w[k][1] = gload4(t.B + bb[k] + 4u * me + 8u);
    }
    const uint32_t xm = me == 0u ? xx[0] : xx[1];
    const uint32_t bm = me == 0u ? bb[0] : bb[1];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        c[k] = 0u;
#pragma unroll
        for (int u = 0; u < 2; ++u)
            c[k] += (uint32_t)(w[k][u].x <= xx[k]) + (uint32_t)(w[k][u].y <= xx[k]) +
                    (uint32_t)(w[k][u].z <= xx[k]) + (uint32_t)(w[k][u].w <= xx[k]);
        c[k] = pair_sum(c[k]);
    }
    const uint32_t cm = me == 0u ? c[0] : c[1];
    uint32_t bit = 0;
    if (lane < nr) {
        bool ok = cm >= 1u;
        if (cm == 16u && bm + 16u < t.m) ok = xm < *glob(t.B + bm + 16u);
        uint32_t j = bm + cm - 1u;
        if (!ok) {
            atomicAdd(t.fallbacks, 1ull);
            j = upper_last(glob(t.B), t.m, xm);
        }
        bit = member_bit(t, v, min(j, t.m - 1));
    }
    return __ballot(bit != 0u);
}

// Membership bits of the addresses in cut /16 blocks by the window PLA, for a
// wave whose 64 lanes are all active.  Unqueued, each address reads its
// 16-boundary window with four 16-byte loads of its own lane, in waves where
// about a third of the lanes need a search, so a wave pays every slot's
// segment search, window loads and compares whichever of its lanes need them.
// Here the addresses that need one are ranked with a ballot and mbcnt and
// queued in a ring in LDS; whenever 64 are waiting, a round (pla_round) gives
// one to every lane, and the round's 64 bits, in queue order, go to two lanes of
// a register, from which each address's lane fetches its own (ds_bpermute) once
// the last, partial round has run.  Queued two slots at a time, 2e8 addresses of
// clustered prefixes took four rounds of 43 busy lanes per iteration; the ring
// takes three, of which two are full (1.50 -> 1.24 ms; 5e8 sessions' labels 3.73
// -> 3.07 ms, with the filter state handed over as it is and the rare load).
template <int N>
__device__ __forceinline__ void pla_window_queued(const DevTable& t, const LdsView& v,
                                                  const uint32_t* a, const uint32_t* st, uint32_t* in) {
    const uint32_t lane = lane_id();
    uint32_t pos[N], head = 0, tail = 0;  // head, tail: wave-uniform
    uint32_t bits = 0;  // lane w: results of the places 32 w .. 32 w + 31
    auto round = [&](uint32_t nr) {
        lds_wave_sync();
        const unsigned long long m = pla_round(t, v, head, nr, lane);
        lds_wave_sync();  // read before the ring's places are written again
        if ((lane & ~1u) == head >> 5) bits = (uint32_t)(m >> (32u * (lane & 1u)));
    };
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const bool nd = st[q] == 2u;
        const unsigned long long m = __ballot(nd);
        pos[q] = tail + rank_in(m);
        if (nd) v.queue[pos[q] & (kPlaQueue - 1u)] = a[q];
        tail += (uint32_t)__popcll(m);
        if (tail - head >= 64u) {
            round(64u);
            head += 64u;
        }
    }
    if (tail != head) round(tail - head);
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const uint32_t w = from_lane(pos[q] >> 5, bits);
        in[q] = st[q] == 2u ? __builtin_amdgcn_ubfe(w, pos[q] & 31u, 1u) : st[q];
    }
}

// Leaf block of each address (the binary search over the LDS sample, or the
// learned model and its bracket), for the kinds whose search ends in a leaf of
// B in global memory.
template <uint32_t KIND, int N>
__device__ __forceinline__ void leaf_blocks(const DevTable& t, const LdsView& v, const uint32_t* a,
                                            uint32_t* b, uint32_t need) {
    if constexpr (KIND == KK_BSEARCH) {
        upper_last_n<N>(v.top, t.n_top, a, b);
    } else if constexpr (KIND == KK_MLP) {
        int p[N];
#pragma unroll
        for (int q = 0; q < N; ++q)
            p[q] = (need >> q) & 1u ? clamp_pos(mlp_predict((const float*)v.w, t.m_f, a[q]), t.m) : 0;
        learned_top_n<N>(t, v, a, p, b, need);
    } else if constexpr (KIND == KK_PLA) {  // a PLA whose bound is too wide for one window
        int p[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            p[q] = 0;
            if (!((need >> q) & 1u)) continue;
            const uint32_t r = a[q] >> (32 - t.radix_bits);
            const uint32_t s0 = radix_entry(v.radix, r), s1 = radix_entry(v.radix, r + 1);
            const uint32_t sg = s0 + upper_last(v.knot + s0, s1 - s0 + 1, a[q]);
            p[q] = clamp_pos(pla_eval(v.knot[sg], v.c[sg], v.g[sg], a[q]), t.m);
        }
        learned_top_n<N>(t, v, a, p, b, need);
    }
}

// Leaves read by pairs of lanes: a wave whose 64 lanes are all active holds up
// to 128 queued addresses x[h] (entry r + 64 h + lane) with their leaf blocks
// b[h].  For each half, two steps of 32 addresses: a pair takes one address per
// step (moved over with ds_bpermute), each of its lanes loads every other
// 16-byte group of the leaf's 16 NL boundaries and counts those <= the address,
// and the pair adds its counts with DPP; every load of a half is issued before
// any is used (a place without an address reads leaf 0, so no load is
// conditional).  The interval is the leaf's first index plus the count minus one
// (the leaf's first boundary is <= the address, as the sample said), exactly
// what the leaf's binary search finds.  The lane at place k of a pair then
// writes the membership bit of its pair's address of step k over the entry.
// Pairs instead of quads halve the steps, whose moves, address arithmetic and
// sums cost more than the further loads (see pla_window_queued).
template <int NL>
__device__ __forceinline__ void leaf_pairs(const DevTable& t, const LdsView& v, const uint32_t* x,
                                           const uint32_t* b, uint32_t r, uint32_t nr,
                                           uint32_t lane) {
    const uint32_t me = lane & 1u, L = t.top_log2;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (64u * h >= nr) break;  // wave-uniform
        const uint32_t nh = min(nr - 64u * h, 64u);  // entries of this half
        uint32_t xx[2], bb[2], c[2];
        uint4 w[2][2 * NL];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const uint32_t src = 32u * k + (lane >> 1);
            xx[k] = from_lane(src, x[h]);
            bb[k] = from_lane(src, b[h]);
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
#pragma unroll
            for (int u = 0; u < 2 * NL; ++u) w[k][u] = gload4(t.B + (bb[k] << L) + 4u * (2 * u + me));
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            uint32_t n = 0;
#pragma unroll
            for (int u = 0; u < 2 * NL; ++u)
                n += (uint32_t)(w[k][u].x <= xx[k]) + (uint32_t)(w[k][u].y <= xx[k]) +
                     (uint32_t)(w[k][u].z <= xx[k]) + (uint32_t)(w[k][u].w <= xx[k]);
            c[k] = pair_sum(n);
        }
        const uint32_t cm = me == 0u ? c[0] : c[1], bm = me == 0u ? bb[0] : bb[1];
        const uint32_t src = 32u * me + (lane >> 1);
        if (src < nh) {
            const uint32_t j = min((bm << L) + cm - 1u, t.m - 1);
            v.queue[r + 64u * h + src] = member_bit(t, v, j);
        }
    }
}

// Interval index of each address (all kinds but SCAN).  Addresses whose bit
// in `need` is clear are skipped (their j is left unspecified); skipped lanes
// issue no memory requests.
template <uint32_t KIND, int N>
__device__ __forceinline__ void intervals(const DevTable& t, const LdsView& v, const uint32_t* a,
                                          uint32_t* j, uint32_t need = 0xFFFFFFFFu) {
    if constexpr (KIND == KK_BSEARCH) {
        upper_last_n<N>(v.top, t.n_top, a, j);
        leaf_search<N>(t, a, j, need);
    } else if constexpr (KIND == KK_TRIE) {
        uint32_t e[N];
#pragma unroll
        for (int q = 0; q < N; ++q) e[q] = (need >> q) & 1u ? *glob(t.trie + (a[q] >> 16)) : 0x80000000u;
#pragma unroll
        for (int q = 0; q < N; ++q)
            if (!(e[q] >> 31)) e[q] = *glob(t.trie + 65536u + e[q] * 256u + ((a[q] >> 8) & 255u));
#pragma unroll
        for (int q = 0; q < N; ++q)
            if (!(e[q] >> 31)) e[q] = *glob(t.trie + 65536u + e[q] * 256u + (a[q] & 255u));
#pragma unroll
        for (int q = 0; q < N; ++q) j[q] = e[q] & 0x7FFFFFFFu;
    } else if constexpr (KIND == KK_PLA) {
        int p[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            p[q] = 0;
            if (!((need >> q) & 1u)) continue;
            // radix bucket -> candidate segments -> last knot <= a
            const uint32_t r = a[q] >> (32 - t.radix_bits);
            const uint32_t s0 = radix_entry(v.radix, r), s1 = radix_entry(v.radix, r + 1);
            const uint32_t s = s0 + upper_last(v.knot + s0, s1 - s0 + 1, a[q]);
            p[q] = clamp_pos(pla_eval(v.knot[s], v.c[s], v.g[s], a[q]), t.m);
        }
        if (t.pla_window) window_search_n<N>(t, a, p, j, need);
        else learned_search_n<N>(t, v, a, p, j, need);
    } else {  // KK_MLP
        int p[N];
#pragma unroll
        for (int q = 0; q < N; ++q)
            p[q] = (need >> q) & 1u ? clamp_pos(mlp_predict((const float*)v.w, t.m_f, a[q]), t.m) : 0;
        learned_search_n<N>(t, v, a, p, j, need);
    }
}

// Algorithm 1 over every row: longest match, lowest row on equal length.
// Returns row + 1, or 0 when no row matches.
__device__ __forceinline__ uint32_t scan_owner(const DevTable& t, const LdsView& v, uint32_t a) {
    uint32_t best = 0, best_len = 0;
    for (uint32_t p = 0; p < t.n_prefix; ++p) {
        uint32_t result = (a & v.mask[p]) - v.cb[p];  // SB - CB
        uint32_t l = v.len[p] + 1;                     // 1..33 so that /0 beats "none"
        bool take = (result == 0u) & (l > best_len);
        best = take ? p + 1 : best;
        best_len = take ? l : best_len;
    }
    return best;
}

// Membership of each address in the union of a scan table's prefixes: the
// parity of the number of its boundaries (in0: an odd start) at or below the
// address, found by a binary search over at most 2^11 of them in LDS, every
// address in lockstep.  They are stored less one, so that b <= a is b - 1 < a,
// padded to 2^steps - 1 words with 0xFFFFFFFF.  Algorithm 1's row scan costs a
// lane 64 x 8 dependent LDS reads for its four sessions against 64 rows, and
// 21 us for the few workgroups of a 10,000-session call; this is 7 rounds of 8
// independent ones.
template <int N>
__device__ __forceinline__ void union_lookup(lds_u32 un, uint32_t steps, uint32_t in0, const uint32_t* a,
                                             uint32_t* in) {
    uint32_t c[N];
#pragma unroll
    for (int q = 0; q < N; ++q) c[q] = 0;
    for (uint32_t h = 1u << steps >> 1; h; h >>= 1) {
#pragma unroll
        for (int q = 0; q < N; ++q) c[q] += un[c[q] + h - 1u] < a[q] ? h : 0u;
    }
#pragma unroll
    for (int q = 0; q < N; ++q) in[q] = (c[q] ^ in0) & 1u;
}

// In/out mark (and, when want_code, the owner code row + 1 or 0) of each
// address.  Label-only lookups first consult the /16 filter: a block that no
// boundary cuts is entirely in or entirely out, which answers most addresses
// from LDS; only addresses in cut blocks run the table's search.
template <uint32_t KIND, int N, int QUEUE = 0>
__device__ __forceinline__ void lookups(const DevTable& t, const LdsView& v, const uint32_t* a,
                                        bool want_code, uint32_t* in, uint32_t* code) {
    if constexpr (KIND == KK_INOUT) {
        inout_lookup<N>((const uint32_t*)v.io, t.io_slot, t.io_list, a, in);
#pragma unroll
        for (int q = 0; q < N; ++q) code[q] = 0;
    } else if constexpr (KIND == KK_UNION) {
        union_lookup<N>(v.io, t.un_steps, t.un_in0, a, in);
#pragma unroll
        for (int q = 0; q < N; ++q) code[q] = 0;
    } else if constexpr (KIND == KK_SCAN) {
#pragma unroll
        for (int q = 0; q < N; ++q) {
            code[q] = scan_owner(t, v, a[q]);
            in[q] = code[q] != 0;
        }
    } else {
        uint32_t need = 0xFFFFFFFFu;
        uint32_t st[N];
        if (!want_code && t.filter_lds) {
            need = 0;
#pragma unroll
            for (int q = 0; q < N; ++q) {
                st[q] = __builtin_amdgcn_ubfe(v.filter[a[q] >> 20], (a[q] >> 15) & 30u, 2u);
                need |= (st[q] == 2u ? 1u : 0u) << q;
            }
        }
        if constexpr ((QUEUE & kQueueWindow) && KIND == KK_PLA) {
            if (v.queue && !want_code && t.filter_lds && t.pla_window && __ballot(1) == ~0ull) {
                pla_window_queued<N>(t, v, a, st, in);
#pragma unroll
                for (int q = 0; q < N; ++q) code[q] = 0;
                return;
            }
        }
        if constexpr ((QUEUE & kQueueSearch) != 0) {
            if (v.queue && !want_code && t.filter_lds && (KIND != KK_PLA || !t.pla_window)) {
                // Wave-level compaction of the searches (section "Coordinated Batch
                // Processing": the chunk is discriminated before the Map stage).  Only
                // addresses in cut /16 blocks need one, about a third of them, yet a
                // wave runs a slot's search whenever any of its lanes needs it.  The
                // addresses that need one are ranked with a ballot and mbcnt per slot,
                // queued in LDS, searched two per active lane per round (dense), and
                // their membership bits read back from their queue entries.  Lanes may
                // be inactive (the ragged last tile, the tail), so the active lanes are
                // ranked among themselves.
                const unsigned long long live = __ballot(1);
                const uint32_t me = rank_in(live);
                const uint32_t n_live = (uint32_t)__popcll(live);
                uint32_t slot[N], cnt = 0;
#pragma unroll
                for (int q = 0; q < N; ++q) {
                    const bool nd = st[q] == 2u;
                    const unsigned long long m = __ballot(nd);
                    slot[q] = cnt + rank_in(m);
                    if (nd) v.queue[slot[q]] = a[q];
                    cnt += (uint32_t)__popcll(m);
                }
                if (cnt) {  // wave-uniform
                    lds_wave_sync();
                    // leaves of 16 or 32 boundaries in global memory, read by pairs
                    // of lanes when the whole wave is active
                    const bool pairs = KIND != KK_TRIE && n_live == 64u && t.n_top > 1 &&
                                       (t.top_log2 == 4 || t.top_log2 == 5);
                    if (pairs) {
                        for (uint32_t r = 0; r < cnt; r += 128) {
                            const uint32_t nr = min(cnt - r, 128u);  // wave-uniform
                            uint32_t x[2] = {me < nr ? v.queue[r + me] : 0u,
                                             me + 64u < nr ? v.queue[r + 64u + me] : 0u};
                            uint32_t b[2] = {0u, 0u};
                            leaf_blocks<KIND, 2>(t, v, x, b,
                                                 (me < nr ? 1u : 0u) | (me + 64u < nr ? 2u : 0u));
                            if (t.top_log2 == 4) leaf_pairs<1>(t, v, x, b, r, nr, me);
                            else leaf_pairs<2>(t, v, x, b, r, nr, me);
                        }
                    }
                    for (uint32_t r = pairs ? cnt : 0u; r < cnt; r += 2 * n_live) {
                        const uint32_t e0 = r + me, e1 = r + n_live + me;
                        uint32_t x[2] = {e0 < cnt ? v.queue[e0] : 0u, e1 < cnt ? v.queue[e1] : 0u};
                        uint32_t j[2] = {0u, 0u};
                        intervals<KIND, 2>(t, v, x, j, (e0 < cnt ? 1u : 0u) | (e1 < cnt ? 2u : 0u));
                        if (e0 < cnt) v.queue[e0] = member_bit(t, v, j[0]);
                        if (e1 < cnt) v.queue[e1] = member_bit(t, v, j[1]);
                    }
                    lds_wave_sync();
#pragma unroll
                    for (int q = 0; q < N; ++q)
                        if (st[q] == 2u) st[q] = v.queue[slot[q]];
                    lds_wave_sync();  // read back before the queue is written again
                }
#pragma unroll
                for (int q = 0; q < N; ++q) {
                    in[q] = st[q];
                    code[q] = 0;
                }
                return;
            }
        }
        if (need) {
            uint32_t j[N];
            intervals<KIND, N>(t, v, a, j, need);
#pragma unroll
            for (int q = 0; q < N; ++q) {
                if (!((need >> q) & 1u)) continue;
                in[q] = member_bit(t, v, j[q]);
                code[q] = want_code ? *glob(t.owner + j[q]) : 0u;
            }
        }
        if (!want_code && t.filter_lds) {
#pragma unroll
            for (int q = 0; q < N; ++q) {
                if (st[q] < 2u) in[q] = st[q];
                code[q] = 0;
            }
        }
    }
}

enum HistMode : int {
    H_NONE = 0,     // labels / institutions / positions only
    H_ATOMIC = 1    // device-scope atomics into the output bins
};

template <int HM>
__device__ __forceinline__ void account(const PassParams& p, uint32_t lab,
                                        uint32_t ts, uint64_t nbytes, Dropped& d) {
    if constexpr (HM == H_NONE) return;
    uint32_t b;
    if (!in_window(p, ts, b)) {
        d.add(lab, nbytes);
        return;
    }
    const uint64_t k = (uint64_t)lab * p.n_bins + b;
    __hip_atomic_fetch_add(p.count + k, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(p.hbytes + k, (unsigned long long)nbytes, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// 16 bytes read once (the columns of a lookup pass): nontemporal loads.  On
// the 1.6e9-session day the in/out lookup pass took 3.08-3.10 ms with plain
// loads and stores and 2.98-2.99 ms with nontemporal loads of src and dst and
// nontemporal label stores (the stores alone: 3.06-3.07 ms).
__device__ __forceinline__ uint4 gload4_nt(const uint32_t* q) {  // q 16-byte aligned
    const u32x4_t v = __builtin_nontemporal_load(glob(reinterpret_cast<const u32x4_t*>(q)));
    return make_uint4(v.x, v.y, v.z, v.w);
}

// Label of session i (scalar path); stores label / institutions when asked.
template <uint32_t KIND, int QUEUE = 0>
__device__ __forceinline__ uint32_t label1(const PassParams& p, const LdsView& v, uint64_t i) {
    const uint32_t a[2] = {*glob(p.src + i), *glob(p.dst + i)};
    const bool wc = p.src_inst != nullptr || p.dst_inst != nullptr;
    uint32_t in[2], code[2];
    lookups<KIND, 2, QUEUE>(p.t, v, a, wc, in, code);
    const uint32_t lab = in[0] | (in[1] << 1);
    if (p.label_out) *glob(p.label_out + i) = (uint8_t)lab;
    if (p.src_inst) *glob(p.src_inst + i) = code[0] ? *glob(p.t.inst + code[0] - 1) : SINET_NO_INST;
    if (p.dst_inst) *glob(p.dst_inst + i) = code[1] ? *glob(p.t.inst + code[1] - 1) : SINET_NO_INST;
    return lab;
}

template <uint32_t KIND, int HM>
__device__ __forceinline__ void one_session(const PassParams& p, const LdsView& v, uint64_t i,
                                            Dropped& d) {
    if (p.pos_out) {
        if constexpr (KIND != KK_SCAN && KIND != KK_LABEL_IN && KIND != KK_INOUT && KIND != KK_UNION) {
            const uint32_t a = p.src[i];
            uint32_t j;
            intervals<KIND, 1>(p.t, v, &a, &j);
            p.pos_out[i] = j;
        }
        return;
    }
    uint32_t lab;
    if constexpr (KIND == KK_LABEL_IN) {
        lab = *glob(p.label_in + i) & 3u;
    } else {
        lab = label1<KIND, HM == H_NONE && queued_kind(KIND) ? kQueueAll : 0>(p, v, i);
    }
    if constexpr (HM != H_NONE) account<HM>(p, lab, *glob(p.ts + i), *glob(p.bytes + i), d);
}

// Labels of four consecutive sessions starting at i from their loaded source
// and destination words (or the given labels); stores labels / institutions
// when asked.
template <uint32_t KIND, int QUEUE = 0>
__device__ __forceinline__ void labels4_from(const PassParams& p, const LdsView& v, uint64_t i,
                                             uint4 s, uint4 t, uint32_t l4, uint32_t lab[4]) {
    if constexpr (KIND == KK_LABEL_IN) {
#pragma unroll
        for (int k = 0; k < 4; ++k) lab[k] = (l4 >> (8 * k)) & 3u;
    } else {
        // sources and destinations of the four sessions, looked up together
        const uint32_t a[8] = {s.x, s.y, s.z, s.w, t.x, t.y, t.z, t.w};
        const bool wc = p.src_inst != nullptr || p.dst_inst != nullptr;
        uint32_t in[8], code[8];
        lookups<KIND, 8, QUEUE>(p.t, v, a, wc, in, code);
        uint32_t sc[4], dc[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            lab[k] = in[k] | (in[4 + k] << 1);
            sc[k] = code[k];
            dc[k] = code[4 + k];
        }
        if (p.label_out) {
            const uint32_t packed = lab[0] | (lab[1] << 8) | (lab[2] << 16) | (lab[3] << 24);
            __builtin_nontemporal_store(packed, glob(reinterpret_cast<uint32_t*>(p.label_out + i)));
        }
        if (p.src_inst) {
            uint4 o;
            o.x = sc[0] ? *glob(p.t.inst + sc[0] - 1) : SINET_NO_INST;
            o.y = sc[1] ? *glob(p.t.inst + sc[1] - 1) : SINET_NO_INST;
            o.z = sc[2] ? *glob(p.t.inst + sc[2] - 1) : SINET_NO_INST;
            o.w = sc[3] ? *glob(p.t.inst + sc[3] - 1) : SINET_NO_INST;
            gstore4(p.src_inst + i, o);
        }
        if (p.dst_inst) {
            uint4 o;
            o.x = dc[0] ? *glob(p.t.inst + dc[0] - 1) : SINET_NO_INST;
            o.y = dc[1] ? *glob(p.t.inst + dc[1] - 1) : SINET_NO_INST;
            o.z = dc[2] ? *glob(p.t.inst + dc[2] - 1) : SINET_NO_INST;
            o.w = dc[3] ? *glob(p.t.inst + dc[3] - 1) : SINET_NO_INST;
            gstore4(p.dst_inst + i, o);
        }
    }
}

template <uint32_t KIND, int QUEUE = 0>
__device__ __forceinline__ void labels4(const PassParams& p, const LdsView& v, uint64_t i,
                                        uint32_t lab[4]) {
    uint4 s = make_uint4(0, 0, 0, 0), t = s;
    uint32_t l4 = 0;
    if constexpr (KIND == KK_LABEL_IN) {
        l4 = *glob(reinterpret_cast<const uint32_t*>(p.label_in + i));
    } else {
        s = gload4(p.src + i);
        t = gload4(p.dst + i);
    }
    labels4_from<KIND, QUEUE>(p, v, i, s, t, l4, lab);
}

template <uint32_t KIND, int HM>
__device__ __forceinline__ void four_sessions(const PassParams& p, const LdsView& v, uint64_t i,
                                            Dropped& d) {
    if (p.pos_out) {
        if constexpr (KIND != KK_SCAN && KIND != KK_LABEL_IN && KIND != KK_INOUT && KIND != KK_UNION) {
            const uint4 a4 = *reinterpret_cast<const uint4*>(p.src + i);
            const uint32_t a[4] = {a4.x, a4.y, a4.z, a4.w};
            uint32_t j[4];
            intervals<KIND, 4>(p.t, v, a, j);
            *reinterpret_cast<uint4*>(p.pos_out + i) = make_uint4(j[0], j[1], j[2], j[3]);
        }
        return;
    }
    uint32_t lab[4];
    labels4<KIND, HM == H_NONE && queued_kind(KIND) ? kQueueAll : 0>(p, v, i, lab);
    if constexpr (HM != H_NONE) {
        const uint4 ts = gload4(p.ts + i);
        const ulonglong2 b01 = gload2(p.bytes + i);
        const ulonglong2 b23 = gload2(p.bytes + i + 2);
        account<HM>(p, lab[0], ts.x, b01.x, d);
        account<HM>(p, lab[1], ts.y, b01.y, d);
        account<HM>(p, lab[2], ts.z, b23.x, d);
        account<HM>(p, lab[3], ts.w, b23.y, d);
    }
}

// Stage the table's hot arrays into LDS (layout chosen on the host).
// Returns the view; *words receives the number of 32-bit words used.
template <uint32_t KIND>
__device__ __forceinline__ LdsView stage_lds(const DevTable& t, uint32_t* lds, uint32_t* words) {
    LdsView v{};
    uint32_t off = 0;
    auto copy = [&](const uint32_t* src, uint32_t n) -> lds_u32 {
        auto* dst = (__attribute__((address_space(3))) uint32_t*)(lds + off);
        for (uint32_t k = threadIdx.x; k < n; k += blockDim.x) dst[k] = *glob(src + k);
        off += n;
        return dst;
    };
    if constexpr (KIND == KK_INOUT) {
        v.io = copy(t.io, t.io_words);
    } else if constexpr (KIND == KK_UNION) {
        v.io = copy(t.un, 1u << t.un_steps);
    } else if constexpr (KIND == KK_SCAN) {
        v.cb = copy(t.cb, t.n_prefix);
        v.mask = copy(t.mask, t.n_prefix);
        v.len = copy(t.len, t.n_prefix);
    } else if constexpr (KIND != KK_LABEL_IN) {
        if (t.filter_lds) v.filter = copy(t.filter, kFilterWords);
        if constexpr (KIND == KK_BSEARCH || KIND == KK_MLP) v.top = copy(t.top, t.n_top);
        if constexpr (KIND == KK_PLA)
            if (!t.pla_window) v.top = copy(t.top, t.n_top);
        if constexpr (KIND == KK_PLA) {
            v.knot = copy(t.knot, t.segments);
            v.c = (lds_f32)copy(reinterpret_cast<const uint32_t*>(t.pla_c), t.segments);
            v.g = (lds_f32)copy(reinterpret_cast<const uint32_t*>(t.pla_g), t.segments);
            v.radix = copy(t.radix, radix_words(t.radix_bits));
        }
        if constexpr (KIND == KK_MLP)
            v.w = (lds_f32)copy(reinterpret_cast<const uint32_t*>(t.mlp), SINET_MLP_PARAMS);
        if (t.lds_member_words) v.member = copy(t.member, t.lds_member_words);
    }
    *words = off;
    __syncthreads();
    return v;
}

// ---------------------------------------------------------------------------
// k_pass: one pass over the sessions.
//   H_NONE    labels / institutions / positions;
//   H_ATOMIC  with far.list: only the sessions the partitioned path flagged
//             as far (see k_stage1), merged with device-scope atomics after
//             the block reduction wrote the bins; without: every session.
// ---------------------------------------------------------------------------
template <uint32_t KIND, int HM, bool VEC>
__device__ __forceinline__ void pass_body(const PassParams& p, const FarList& far) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    uint32_t used = 0;
    if (HM == H_ATOMIC && far.list && *glob(far.count) == 0) return;  // before the table is staged
    LdsView v = stage_lds<KIND>(p.t, lds, &used);
    if constexpr (HM == H_NONE && queued_kind(KIND)) {
        if (p.queue_words) v.queue = (__attribute__((address_space(3))) uint32_t*)(lds + used + (threadIdx.x >> 6) * p.queue_words);
    }
    Dropped d{};
    if (HM == H_ATOMIC && far.list) {
        const uint32_t nfar = *far.count;
        for (uint32_t q = blockIdx.x; q < nfar; q += gridDim.x) {
            const uint64_t c = far.list[q];
            for (uint32_t s = threadIdx.x; s < kChunk; s += blockDim.x) {
                const uint64_t i = c * kChunk + s;
                if (i < p.n && ((far.bits[c * (kChunk / 32) + s / 32] >> (s & 31)) & 1u))
                    one_session<KIND, HM>(p, v, i, d);
            }
        }
    } else {
        // XCD-contiguous split of the tiles (one tile = 4 sessions per lane).
        const uint64_t groups = (p.n + 3) / 4;
        const uint64_t tile = blockDim.x;
        const uint64_t n_tiles = (groups + tile - 1) / tile;
        const uint32_t W = gridDim.x;
        const uint32_t xcd = blockIdx.x % kXcds;
        const uint32_t lid = blockIdx.x / kXcds;
        const uint32_t per = W / kXcds, rem = W % kXcds;
        const uint32_t nx = per + (xcd < rem ? 1u : 0u);
        const uint64_t cum = (uint64_t)xcd * per + min(xcd, rem);
        const uint64_t T0 = n_tiles * cum / W;
        const uint64_t T1 = n_tiles * (cum + nx) / W;
        if constexpr (HM == H_NONE && VEC && KIND != KK_LABEL_IN) {
            if (!p.pos_out) {
                // labels / institutions only: the next tile's addresses are
                // loaded before the current tile's lookups run
                auto full = [&](uint64_t tl) { return (tl * tile + threadIdx.x) * 4 + 4 <= p.n; };
                uint4 cs = make_uint4(0, 0, 0, 0), cd = cs, ns = cs, nd = cs;
                uint64_t tl = T0 + lid;
                if (tl < T1 && full(tl)) {
                    const uint64_t i = (tl * tile + threadIdx.x) * 4;
                    cs = gload4_nt(p.src + i);
                    cd = gload4_nt(p.dst + i);
                }
                for (; tl < T1; tl += nx) {
                    const uint64_t tn = tl + nx;
                    if (tn < T1 && full(tn)) {
                        const uint64_t i = (tn * tile + threadIdx.x) * 4;
                        ns = gload4_nt(p.src + i);
                        nd = gload4_nt(p.dst + i);
                    }
                    const uint64_t g = tl * tile + threadIdx.x;
                    if (full(tl)) {
                        uint32_t lab[4];
                        constexpr int kQ = HM == H_NONE && queued_kind(KIND) ? kQueueAll : 0;
                        labels4_from<KIND, kQ>(p, v, g * 4, cs, cd, 0u, lab);
                    } else if (g * 4 < p.n) {
                        for (uint64_t i = g * 4; i < p.n && i < g * 4 + 4; ++i)
                            one_session<KIND, HM>(p, v, i, d);
                    }
                    cs = ns;
                    cd = nd;
                }
                return;
            }
        }
        for (uint64_t tl = T0 + lid; tl < T1; tl += nx) {
            const uint64_t g = tl * tile + threadIdx.x;
            if (g >= groups) continue;
            if (VEC && g * 4 + 4 <= p.n) {
                four_sessions<KIND, HM>(p, v, g * 4, d);
            } else {
                for (uint64_t i = g * 4; i < p.n && i < g * 4 + 4; ++i)
                    one_session<KIND, HM>(p, v, i, d);
            }
        }
    }
    if constexpr (HM != H_NONE) d.flush(p.dropped);
}

template <uint32_t KIND, int HM, bool VEC>
__global__ void __launch_bounds__(kMaxBlock) k_pass(PassParams p, FarList far) {
    pass_body<KIND, HM, VEC>(p, far);
}

// The label pass over the in/out index (the plain form's lookup): its 64 KB
// of LDS lets two 1024-lane workgroups share a CU once the kernel fits in 64
// VGPRs (eight waves per SIMD), twice the waves to hide the column loads.
__global__ void __launch_bounds__(kMaxBlock) __attribute__((amdgpu_waves_per_eu(8)))
k_pass_inout(PassParams p, FarList far) {
    pass_body<KK_INOUT, H_NONE, true>(p, far);
}

// ---------------------------------------------------------------------------
// Partitioned histogram: the two-stage map-reduce, both stages on the GPU.
//
// Stage 1 (k_stage1, fused with discrimination): a workgroup takes a chunk of
// kChunk consecutive sessions, labels them and maps each in-window session to
// (block = bin / kBlockBins, offset, label).  Sessions are counting-sorted in
// LDS by block relative to the chunk's first block (a window of kWin blocks)
// and written as 4-byte records, grouped by block, into the chunk's own slot
// range (every block's segment padded with null records to whole 16-byte
// groups); the chunk's directory lists (block, first slot, slots) for every
// block it touched.  Near time-sorted input (the paper's session logs)
// touches few blocks per chunk.
// Segment index: per-block directory counts, an exclusive scan, and a fill
// that groups the directory entries by block (k_fill).
// Stage 2 (k_stage2): persistent workgroups take blocks in turn, accumulate a
// block's segments' records in LDS and write the block's count and byte bins
// once, with coalesced stores, while the next block's segment list is in
// flight; no zero-fill and no global atomics.
// Far path: a session outside its chunk's block window, with bytes >= 2^52,
// or beyond the chunk's extra record slots is flagged and merged afterwards
// by k_pass<H_ATOMIC> with global atomics, so any input stays exact.
//
// Record (self-contained, so stage 2 needs no other read):
//   label (2 bits) | offset in block (10) | 0 | byte count (19)   if bytes < 2^19
//   label (2 bits) | offset in block (10) | 1 | part k (2) | bits 17k..17k+16
//                                              of the byte count  otherwise,
// one record per 17-bit part up to the highest nonzero one (2 to 4 records);
// part 0 carries the session's count.  0xFFFFFFFF is the null record (a part 3
// holds at most bit 51, so no real record has that value).
// ---------------------------------------------------------------------------
// Raw column words of one lane's four sessions (loaded one chunk ahead).
struct Raw4 {
    uint4 src, dst, ts;
    ulonglong2 b01, b23;
    uint32_t l4;
};

template <uint32_t KIND>
__device__ __forceinline__ void load4(const PassParams& p, uint64_t i, Raw4& r) {
    if constexpr (KIND == KK_LABEL_IN) {
        r.l4 = *glob(reinterpret_cast<const uint32_t*>(p.label_in + i));
    } else {
        r.src = gload4(p.src + i);
        r.dst = gload4(p.dst + i);
    }
    r.ts = gload4(p.ts + i);
    r.b01 = gload2(p.bytes + i);
    r.b23 = gload2(p.bytes + i + 2);
}

// LDS scratch of one stage-1 workgroup.
struct Stage1Shared {
    uint32_t cnt[kWin];
    uint32_t base[kWin];
    uint32_t far[kChunk / 32];
    uint32_t wmin[kStage1Block / 64];
    uint32_t nextra, nfar;
};
// Static LDS of a stage-1 workgroup: two alternating Stage1Shared and the
// record buffer (one suffices: a chunk fills it only after its first barrier,
// which every lane reaches after copying the previous chunk out).
constexpr size_t kStage1StaticLds = 2 * sizeof(Stage1Shared) + sizeof(uint4) * (kChunkSlots / 4);

// Records of one session's byte count (see the record format above).
__device__ __forceinline__ uint32_t record_parts(unsigned long long by) {
    if (by < kSmallMax) return 1u;
    return by < (1ull << 34) ? 2u : (by < (1ull << 51) ? 3u : 4u);
}

// Stage 1 on one chunk.  c is the chunk within the stream (sessions
// c * kChunk + ...), g its index in the workspace (slots, directory, far
// bits) and b0 the workspace index of the stream's first block.
template <uint32_t KIND>
__device__ __forceinline__ void stage1_chunk(const PassParams& p, const PartWs& w, const LdsView& v,
                                             Stage1Shared& sh, uint4* srec, uint64_t c, uint64_t g, uint32_t b0,
                                             const Raw4& cur, bool full, Dropped& d) {
    const uint32_t tid = threadIdx.x;
    const uint64_t i0 = c * kChunk + (uint64_t)tid * 4;
    uint32_t lab[4], ts[4], bin[4];
    unsigned long long by[4];
    bool inw[4];
    if (full) {
        labels4_from<KIND>(p, v, i0, cur.src, cur.dst, cur.l4, lab);
        ts[0] = cur.ts.x; ts[1] = cur.ts.y; ts[2] = cur.ts.z; ts[3] = cur.ts.w;
        by[0] = cur.b01.x; by[1] = cur.b01.y; by[2] = cur.b23.x; by[3] = cur.b23.y;
#pragma unroll
        for (int k = 0; k < 4; ++k) inw[k] = in_window(p, ts[k], bin[k]);
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint64_t i = i0 + k;
            inw[k] = false;
            lab[k] = 0;
            ts[k] = 0;
            by[k] = 0;
            bin[k] = 0;
            if (i < p.n) {
                if constexpr (KIND == KK_LABEL_IN) {
                    lab[k] = *glob(p.label_in + i) & 3u;
                } else {
                    lab[k] = label1<KIND>(p, v, i);
                }
                ts[k] = *glob(p.ts + i);
                by[k] = *glob(p.bytes + i);
                inw[k] = in_window(p, ts[k], bin[k]);
            }
        }
    }
    uint32_t blk[4];
    uint32_t mymin = 0xFFFFFFFFu;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        blk[k] = bin[k] / kBlockBins;
        if (inw[k]) mymin = min(mymin, blk[k]);
        else if (i0 + k < p.n) d.add(lab[k], by[k]);
    }
    // sh alternates between two buffers from chunk to chunk, so clearing this
    // chunk's counters cannot race with lanes still writing the previous one
    mymin = wave_min(mymin);
    if ((tid & 63) == 0) sh.wmin[tid >> 6] = mymin;
    if (tid < kWin) sh.cnt[tid] = 0;
    for (uint32_t k = tid; k < kChunk / 32; k += kStage1Block) sh.far[k] = 0;
    if (tid == 0) {
        sh.nextra = 0;
        sh.nfar = 0;
    }
    __syncthreads();
    uint32_t bmin = 0xFFFFFFFFu;
#pragma unroll
    for (int k = 0; k < kStage1Block / 64; ++k) bmin = min(bmin, sh.wmin[k]);
    uint32_t rank[4], nrec[4];
    bool loc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t r = blk[k] - bmin;
        loc[k] = inw[k] && r < kWin && by[k] < (1ull << 52);
        nrec[k] = record_parts(by[k]);
        if (loc[k] && nrec[k] > 1u) {
            const uint32_t e = atomicAdd(&sh.nextra, nrec[k] - 1u);
            if (e + nrec[k] - 1u > (uint32_t)kExtraRecs) loc[k] = false;
        }
        rank[k] = loc[k] ? atomicAdd(&sh.cnt[r], nrec[k]) : 0u;
        if (inw[k] && !loc[k]) {
            const uint32_t sidx = tid * 4 + k;
            atomicOr(&sh.far[sidx >> 5], 1u << (sidx & 31));
            atomicAdd(&sh.nfar, 1u);
        }
    }
    __syncthreads();
    if (tid < 64) {  // exclusive scan of the kWin (= 64) padded block counts, one wave
        const uint32_t x = (sh.cnt[tid] + 3u) & ~3u;
        uint32_t inc = x;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)inc, o);
            if ((int)tid >= o) inc += y;
        }
        sh.base[tid] = inc - x;
        // null records in the padding of the block's segment
        uint32_t* lpad = reinterpret_cast<uint32_t*>(srec);
        for (uint32_t q = inc - x + sh.cnt[tid]; q < inc; ++q) lpad[q] = 0xFFFFFFFFu;
        // directory entry of every touched block
        const bool nz = x != 0;
        const unsigned long long m = __ballot(nz);
        const uint32_t e = __popcll(m & ((1ull << tid) - 1ull));
        if (nz) {
            const uint32_t b = b0 + bmin + tid;
            w.dir[g * kWin + e] = make_uint4(b, (uint32_t)(g * kChunkSlots) + (inc - x), x, 0u);
            atomicAdd(w.seg_count + b, 1u);
        }
        if (tid == 0) w.nd[g] = (uint32_t)__popcll(m);
    }
    __syncthreads();
    uint32_t* lrec = reinterpret_cast<uint32_t*>(srec);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (!loc[k]) continue;
        const uint32_t r = blk[k] - bmin;
        const uint32_t off = bin[k] - blk[k] * kBlockBins;
        const uint32_t key = (lab[k] << 30) | (off << 20);
        const uint32_t at = sh.base[r] + rank[k];
        if (nrec[k] == 1u) {
            lrec[at] = key | (uint32_t)by[k];
        } else {
            for (uint32_t q = 0; q < nrec[k]; ++q)
                lrec[at + q] = key | (1u << 19) | (q << 17) | (uint32_t)((by[k] >> (17 * q)) & 0x1FFFFu);
        }
    }
    __syncthreads();
    {   // the filled slots of the chunk, one 16-byte store per lane
        const uint32_t nloc = sh.base[kWin - 1] + ((sh.cnt[kWin - 1] + 3u) & ~3u);
        uint4* dst = reinterpret_cast<uint4*>(w.rec + g * kChunkSlots);
        for (uint32_t k = tid; k < nloc / 4; k += kStage1Block) dst[k] = srec[k];
    }
    if (sh.nfar) {
        for (uint32_t k = tid; k < kChunk / 32; k += kStage1Block)
            w.farbits[g * (kChunk / 32) + k] = sh.far[k];
        if (tid == 0) w.farlist[atomicAdd(w.farcount, 1u)] = (uint32_t)g;
    }
}

template <uint32_t KIND>
__global__ void __launch_bounds__(kStage1Block, 4) k_stage1(PassParams p, PartWs w) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    __shared__ Stage1Shared sh[2];
    __shared__ uint4 srec[kChunkSlots / 4];
    __shared__ uint32_t s_run;
    if (w.gate && !*glob(w.gate)) return;
    uint32_t used = 0;
    const LdsView v = stage_lds<KIND>(p.t, lds, &used);
    Dropped d{};
    const uint32_t tid = threadIdx.x;
    const uint64_t n_chunks = w.n_chunks;
    uint32_t iter = 0;
    // a chunk is "full" when its kChunk sessions exist and vector loads are allowed
    auto full = [&](uint64_t c) { return w.vec && (c + 1) * kChunk <= p.n; };
    // workgroups take runs of consecutive chunks from a counter, so
    // one that falls behind (a busy XCD, a chunk of far sessions) takes fewer;
    // every lane reads s_run before the chunk's first barrier, tid 0 writes it
    // again only after the run's last one
    for (;;) {
        if (tid == 0) s_run = atomicAdd(w.next_run, 1u);
        __syncthreads();
        const uint64_t c0 = (uint64_t)__builtin_amdgcn_readfirstlane((int)s_run) * w.run;
        if (c0 >= n_chunks) break;
        const uint64_t c1 = c0 + w.run < n_chunks ? c0 + w.run : n_chunks;
        Raw4 cur{}, nxt{};
        if (full(c0)) load4<KIND>(p, c0 * kChunk + (uint64_t)tid * 4, cur);
        for (uint64_t c = c0; c < c1; ++c) {
            if (c + 1 < c1 && full(c + 1)) load4<KIND>(p, (c + 1) * kChunk + (uint64_t)tid * 4, nxt);
            stage1_chunk<KIND>(p, w, v, sh[iter++ & 1u], srec, c, c, 0u, cur, full(c), d);
            cur = nxt;
        }
    }
    d.flush(p.dropped);
}

// ---------------------------------------------------------------------------
// k_local: the reduce of coarse bins (many sessions per bin), one pass with the
// labels computed or given.
//
// Session logs are nearly sorted by time, so with many sessions per bin the
// sessions of a contiguous range touch few bins.  A workgroup takes one range
// and walks it in runs of at most 2^17 - 1 sessions; during a run it keeps a
// window of `bins` bins x 4 labels in LDS, one 64-bit word each (count << 47 |
// byte sum), adds every session with one LDS atomic, and at the run's end adds
// the words that are not zero to the (cleared) output with device atomics and
// places the window anew.  When all bins fit, the window is the histogram.
// Sessions outside the window or with 2^30 bytes or more go to the output
// directly, so any input is exact.  With 2^reps copies of the window, lane l
// using copy l % 2^reps, lanes that hit the same bin (coarse bins: a wave's
// sessions share one or two) meet in fewer words.
//
// HBM bound: 12 B/session (and 8 B of addresses, or 1 B of labels).  A step
// needs no barrier; runs do, two each.  Measured against the records (whose
// stage 2 has one workgroup per 1,024 bins, and whose counters a few blocks
// contend for) and, from 2^28 sessions on, the sliding window (whose 5-bit
// counts overflowed into one event list then): 1e8 sessions of a day into 86,400
// one-second bins, lookups included, 1.78 -> 0.38 ms (5.3 TB/s); into 1,440
// minutes 89.7 -> 0.37 ms; 4e8 labelled sessions into 86,400 seconds 63.4 ->
// 0.91 ms (5.7 TB/s), into 144 ten-minute frames (before: 32-bit count and
// 64-bit byte atomics on one copy) 1.65 -> 0.88 ms (5.9 TB/s).
// ---------------------------------------------------------------------------
constexpr uint32_t kLocalShift = 47;                       // window word: count << 47 | bytes
constexpr uint64_t kLocalMaxBytes = 1ull << 30;            // larger counts go to the output
static_assert((kLocalMaxBytes - 1) * kLocalRun < (1ull << kLocalShift), "no carry into the count");

// Runs out of order (see local_defer): records by block of kBlockBins bins.  The
// kernels derive it from its base, since scalar registers are short in k_local.
struct DeferWs {
    uint32_t* any;     // nonzero: some run's sessions are here
    uint32_t* on;      // [steps] the step's sessions are here
    uint32_t* dir;     // [blocks][steps] the step's records of a block: first slot | slots << 16
    uint32_t* rec;     // [steps][kDeferSlots] records (their format is stage 1's)
    uint32_t steps, blocks;
};

constexpr uint32_t kDeferBlocks = kDeferMaxBins / kBlockBins;
constexpr uint32_t kDeferExtra = 768;  // records beyond one per session a step may hold
constexpr uint32_t kDeferSlots = 4 * kMaxBlock + kDeferExtra + 3 * kDeferBlocks;
static_assert(kDeferBlocks == 64, "a wave scans their counts");
static_assert(kDeferSlots % 4 == 0 && kDeferSlots < (1u << 16), "whole groups, 16-bit slots");

__host__ __device__ inline DeferWs defer_at(uint32_t* base, uint64_t n, uint32_t n_bins) {
    DeferWs d;
    d.steps = (uint32_t)((n + 4 * kMaxBlock - 1) / (4 * kMaxBlock));
    d.blocks = (n_bins + kBlockBins - 1) / kBlockBins;
    const uint32_t lines = (d.steps + 31u) & ~31u;
    d.any = base;
    d.on = base + 32;
    d.dir = d.on + lines;
    d.rec = d.dir + (uint64_t)lines * d.blocks;
    return d;
}

struct LocalArgs {
    uint32_t bins;     // bins of the window
    uint32_t reps;     // log2 of the window's copies
    uint32_t run;      // steps of a run
    uint32_t whole;    // the window is the whole histogram
    const uint32_t* gate;  // NULL, or a word: nonzero when another reduce runs instead
    uint32_t* aside;   // k_local's third form only: base of the DeferWs
};

// A workgroup's window: `bins` bins from w0 on, 2^reps copies.
struct LocalWin {
    unsigned long long* h;
    uint32_t bins, reps, w0;
};

// First bin of the next window: a sixteenth of it before the median of the
// waves' first bins (a few stray sessions do not move it).  m: this lane's first
// bin, ~0 for none.  Called by the whole workgroup; s_min holds a word per wave.
__device__ __forceinline__ uint32_t local_place(uint32_t m, uint32_t bins, uint32_t* s_min) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    m = wave_min(m);
    if (lane == 0) s_min[wave] = m;
    lds_barrier();
    const uint32_t mine = lane < nw ? s_min[lane] : 0xFFFFFFFFu;
    const uint32_t valid = (uint32_t)__popcll(__ballot(mine != 0xFFFFFFFFu));
    uint32_t rank = 0;
    for (uint32_t k = 0; k < nw; ++k) {
        const uint32_t o = s_min[k];
        rank += (o < mine || (o == mine && k < lane)) ? 1u : 0u;
    }
    const unsigned long long at = __ballot(mine != 0xFFFFFFFFu && rank == valid / 2);
    const uint32_t med = at ? (uint32_t)__builtin_amdgcn_readlane((int)mine, __builtin_ctzll(at)) : 0u;
    return med > bins / 16u ? med - bins / 16u : 0u;
}

// One session into the window (copy rep), the output or the dropped counters.
__device__ __forceinline__ void local_add(const PassParams& p, const LocalWin& w, uint32_t rep, uint32_t lab,
                                          uint32_t ts, unsigned long long by, Dropped& d) {
    uint32_t bin;
    const bool inw = in_window(p, ts, bin);
    const uint32_t off = bin - w.w0;
    if (inw && off < w.bins && by < kLocalMaxBytes) {
        atomicAdd(&w.h[((off * 4u + lab) << w.reps) + rep], (1ull << kLocalShift) | by);
    } else if (inw) {
        const uint64_t x = (uint64_t)lab * p.n_bins + bin;
        __hip_atomic_fetch_add(p.count + x, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(p.hbytes + x, by, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        d.add(lab, by);
    }
}

// The lane's four sessions from i0 on: loaded ones (full), or those below n
// (bit k of the result: session k).
template <uint32_t KIND>
__device__ __forceinline__ uint32_t local_get4(const PassParams& p, const LdsView& v, uint64_t i0,
                                               const Raw4& cur, bool full, uint32_t* lab, uint32_t* ts,
                                               unsigned long long* by) {
    if (full) {
        labels4_from<KIND>(p, v, i0, cur.src, cur.dst, cur.l4, lab);
        ts[0] = cur.ts.x; ts[1] = cur.ts.y; ts[2] = cur.ts.z; ts[3] = cur.ts.w;
        by[0] = cur.b01.x; by[1] = cur.b01.y; by[2] = cur.b23.x; by[3] = cur.b23.y;
        return 15u;
    }
    uint32_t has = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint64_t i = i0 + k;
        lab[k] = ts[k] = 0;
        by[k] = 0;
        if (i >= p.n) continue;
        has |= 1u << k;
        if constexpr (KIND == KK_LABEL_IN) lab[k] = *glob(p.label_in + i) & 3u;
        else lab[k] = label1<KIND>(p, v, i);
        ts[k] = *glob(p.ts + i);
        by[k] = *glob(p.bytes + i);
    }
    return has;
}

// They go into the window.
template <uint32_t KIND>
__device__ __forceinline__ void local_add4(const PassParams& p, const LdsView& v, const LocalWin& w,
                                           uint32_t rep, uint64_t i0, const Raw4& cur, bool full, Dropped& d) {
    uint32_t lab[4], ts[4];
    unsigned long long by[4];
    const uint32_t has = local_get4<KIND>(p, v, i0, cur, full, lab, ts, by);
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if ((has >> k) & 1u) local_add(p, w, rep, lab[k], ts[k], by[k], d);
}

// First bin of the lane's four sessions (~0: none in the histogram).
__device__ __forceinline__ uint32_t local_first(const PassParams& p, uint64_t i0, const Raw4& cur, bool full) {
    const uint32_t t4[4] = {cur.ts.x, cur.ts.y, cur.ts.z, cur.ts.w};
    uint32_t m = 0xFFFFFFFFu;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool has = full || i0 + k < p.n;
        const uint32_t ts = full ? t4[k] : (has ? *glob(p.ts + i0 + k) : 0u);
        uint32_t bin;
        if (has && in_window(p, ts, bin)) m = min(m, bin);
    }
    return m;
}

// The window's words added to the output and cleared; consecutive lanes take
// consecutive bins of a label, as the output does.  Between barriers.
__device__ __forceinline__ void local_flush(const PassParams& p, const LocalWin& w) {
    for (uint32_t k = threadIdx.x; k < 4u * w.bins; k += blockDim.x) {
        const uint32_t l = k / w.bins, b = k - l * w.bins;
        unsigned long long c = 0, y = 0;
        for (uint32_t r = 0; r < 1u << w.reps; ++r) {
            unsigned long long* e = &w.h[((b * 4u + l) << w.reps) + r];
            const unsigned long long x = *e;
            if (x) *e = 0;
            c += x >> kLocalShift;
            y += x & ((1ull << kLocalShift) - 1ull);
        }
        if (c) {
            const uint64_t x = (uint64_t)l * p.n_bins + w.w0 + b;
            __hip_atomic_fetch_add(p.count + x, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_fetch_add(p.hbytes + x, y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// ---- runs out of order -------------------------------------------------------
// A session outside the window costs two device atomics, 35 times one inside it,
// and input in no order has nearly all outside.  So, for the calls that the third
// form of k_local takes, a run first tries 64 of its sessions, evenly spaced (a
// line each: 1,024 of them cost 8 % of the call's time); where more than an eighth
// would miss the window, it leaves its sessions to k_aside, which writes them as
// records grouped by block of bins, and k_deferred, which adds those up block by
// block (both return at once when there are none).  Sessions that the records
// cannot take (2^52 bytes or more, or a step with many large byte counts) go to
// the output directly.  (Writing the records inside k_local instead saves a launch,
// but spills registers in the loop of the runs in order: 371 -> 430 us for 1e8
// sessions looked up in the in/out index.)
//
// 1e8 shuffled labelled sessions: into 65,536 bins 8.37 -> 0.65 ms (the two-stage
// records 4.80, whose stage 2 has one workgroup per block), into 6,000 8.6 -> 0.53
// (7.40); looked up, into 43,200 8.63 -> 0.79.  In order 0.240 -> 0.250 ms, looked
// up 0.372 -> 0.382: the room for the records (a gap of 6 us in the stream where
// it is given back) and the launches that find nothing to do.  The first call
// after memory was freed otherwise (a table destroyed) maps that room again, 66 us
// for 1e8 sessions, 150 to 200 for 2e8; taking it while k_local runs, with the flags
// of the runs in an allocation of their own, saved that but cost every call a second
// gap (2e8 looked up 886 -> 895 us), and so did a k_aside that found the runs
// out of order itself (10 us, the samples' reads).

// Whether more than an eighth of the bins that the lanes with `counts` bring lie
// outside the window.  Called by the whole workgroup; s_vote holds a word per wave.
__device__ __forceinline__ bool local_strays(const LocalWin& w, uint32_t bin, bool counts, uint32_t* s_vote) {
    const uint32_t lane = threadIdx.x & 63u, nw = blockDim.x >> 6;
    const uint32_t in = (uint32_t)__popcll(__ballot(counts));
    const uint32_t miss = (uint32_t)__popcll(__ballot(counts && bin - w.w0 >= w.bins));
    if (lane == 0) s_vote[threadIdx.x >> 6] = miss << 16 | in;
    lds_barrier();
    uint32_t sum = 0;
    for (uint32_t k = 0; k < nw; ++k) sum += s_vote[k];
    return (sum >> 16) * 8u > (sum & 0xFFFFu);
}

// Its third form (DEFER, 1,024 lanes) sets runs out of order aside.
template <uint32_t KIND, bool VEC, bool DEFER>
__global__ void __launch_bounds__(kMaxBlock) k_local(PassParams p, LocalArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    __shared__ uint32_t s_min[kMaxBlock / 64], s_vote[DEFER ? kMaxBlock / 64 : 1];
    if (a.gate && *glob(a.gate)) return;
    uint32_t used = 0;
    const LdsView v = stage_lds<KIND>(p.t, lds, &used);
    LocalWin w{reinterpret_cast<unsigned long long*>(lds + ((used + 3) & ~3u)), a.bins, a.reps, 0u};
    const uint32_t tid = threadIdx.x;
    for (uint32_t k = tid; k < a.bins * 4u << a.reps; k += blockDim.x) w.h[k] = 0;
    const uint32_t rep = tid & ((1u << a.reps) - 1u);
    Dropped d{};
    const uint64_t step = 4ull * blockDim.x;
    const uint64_t n_steps = (p.n + step - 1) / step;
    const uint64_t s0 = n_steps * blockIdx.x / gridDim.x, s1 = n_steps * (blockIdx.x + 1) / gridDim.x;
    auto full = [&](uint64_t s) { return VEC && (s + 1) * step <= p.n; };
    // every 16th lane's sample of the run from step r0 on
    const bool tries = (tid & 15u) == 0;
    auto sample = [&](uint64_t r0) -> uint32_t {
        if (r0 >= s1 || !tries) return 0u;
        const uint64_t i0 = r0 * step, i1 = min(p.n, min(r0 + a.run, s1) * step);
        return *glob(p.ts + i0 + (i1 - i0) * tid / blockDim.x);
    };
    Raw4 cur{}, nxt{};
    if (s0 < s1 && full(s0)) load4<KIND>(p, s0 * step + 4ull * tid, cur);
    __syncthreads();
    for (uint64_t r0 = s0; r0 < s1; r0 += a.run) {
        const uint64_t r1 = r0 + a.run < s1 ? r0 + a.run : s1;
        uint32_t tried = 0;
        if constexpr (DEFER) tried = sample(r0);
        if (!a.whole) w.w0 = local_place(local_first(p, r0 * step + 4ull * tid, cur, full(r0)), a.bins, s_min);
        if constexpr (DEFER) {
            uint32_t bin;
            const bool counts = in_window(p, tried, bin) && tries;
            const bool aside = local_strays(w, bin, counts, s_vote);
            if (tid < r1 - r0) *glob(defer_at(a.aside, p.n, p.n_bins).on + r0 + tid) = aside ? 1u : 0u;
            if (aside) {  // k_aside's
                if (tid == 0) *glob(a.aside) = 1u;
                if (r1 < s1 && full(r1)) load4<KIND>(p, r1 * step + 4ull * tid, cur);
                continue;
            }
        }
        for (uint64_t s = r0; s < r1; ++s) {
            if (s + 1 < s1 && full(s + 1)) load4<KIND>(p, (s + 1) * step + 4ull * tid, nxt);
            local_add4<KIND>(p, v, w, rep, s * step + 4ull * tid, cur, full(s), d);
            cur = nxt;
        }
        lds_barrier();
        local_flush(p, w);
        lds_barrier();
    }
    d.flush(p.dropped);
}

// LDS of a step of records.
struct DeferShared {
    uint4 rec[kDeferSlots / 4];
    uint32_t cnt[kDeferBlocks], base[kDeferBlocks];
    uint32_t extra, slots, pad[2];
};

// The steps (of 4,096 sessions) that k_local set aside, as records grouped by
// block of bins.
template <uint32_t KIND, bool VEC>
__global__ void __launch_bounds__(kMaxBlock) k_aside(PassParams p, uint32_t* aside) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    __shared__ DeferShared sh;
    if (*glob(aside) == 0) return;
    uint32_t used = 0;
    const LdsView v = stage_lds<KIND>(p.t, lds, &used);
    const DeferWs w = defer_at(aside, p.n, p.n_bins);
    const uint32_t tid = threadIdx.x;
    uint32_t* lrec = reinterpret_cast<uint32_t*>(sh.rec);
    Dropped d{};
    for (uint64_t s = blockIdx.x; s < w.steps; s += gridDim.x) {
        if (*glob(w.on + s) == 0) continue;
        const uint64_t i0 = s * (4 * kMaxBlock) + 4ull * tid;
        const bool full = VEC && (s + 1) * (4 * kMaxBlock) <= p.n;
        Raw4 raw{};
        if (full) load4<KIND>(p, i0, raw);
        uint32_t lab[4], ts[4], bin[4], rank[4];
        unsigned long long by[4];
        if (tid < kDeferBlocks) sh.cnt[tid] = 0;  // last read before the previous step's last barrier
        if (tid == 0) sh.extra = 0;
        lds_barrier();
        const uint32_t has = local_get4<KIND>(p, v, i0, raw, full, lab, ts, by);
        uint32_t rec = 0;  // bit k: session k becomes records
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            rank[k] = 0;
            const bool inw = in_window(p, ts[k], bin[k]);
            if (!((has >> k) & 1u)) continue;
            if (!inw) {
                d.add(lab[k], by[k]);
                continue;
            }
            const uint32_t more = record_parts(by[k]) - 1u;
            bool fits = by[k] < (1ull << 52);
            if (fits && more) fits = atomicAdd(&sh.extra, more) + more <= kDeferExtra;
            if (fits) {
                rec |= 1u << k;
                rank[k] = atomicAdd(&sh.cnt[bin[k] / kBlockBins], more + 1u);
            } else {
                const uint64_t x = (uint64_t)lab[k] * p.n_bins + bin[k];
                __hip_atomic_fetch_add(p.count + x, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_fetch_add(p.hbytes + x, by[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        lds_barrier();
        if (tid < 64) {  // places of the blocks' groups, each padded to whole 16 bytes
            const uint32_t c = sh.cnt[tid], x = (c + 3u) & ~3u;
            uint32_t inc = x;
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t y = (uint32_t)__shfl_up((int)inc, o);
                if ((int)tid >= o) inc += y;
            }
            sh.base[tid] = inc - x;
            for (uint32_t q = inc - x + c; q < inc; ++q) lrec[q] = 0xFFFFFFFFu;
            if (tid < w.blocks) *glob(w.dir + (uint64_t)tid * w.steps + s) = (inc - x) | x << 16;
            if (tid == 63) sh.slots = inc;
        }
        lds_barrier();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (!((rec >> k) & 1u)) continue;
            const uint32_t blk = bin[k] / kBlockBins, key = lab[k] << 30 | (bin[k] - blk * kBlockBins) << 20;
            const uint32_t at = sh.base[blk] + rank[k], parts = record_parts(by[k]);
            if (parts == 1u) {
                lrec[at] = key | (uint32_t)by[k];
            } else {
                for (uint32_t q = 0; q < parts; ++q)
                    lrec[at + q] = key | 1u << 19 | q << 17 | ((uint32_t)(by[k] >> (17 * q)) & 0x1FFFFu);
            }
        }
        lds_barrier();
        uint32_t* dst = w.rec + s * kDeferSlots;
        for (uint32_t k = tid; k < sh.slots / 4; k += kMaxBlock) gstore4(dst + 4 * k, sh.rec[k]);
    }
    d.flush(p.dropped);
}

// Exclusive scan of n u32 counts into out[0..n] (out[n] = total), in three
// launches: per-tile sums, a single-workgroup scan of the tile sums, and the
// per-tile rescan.  kScanTile elements per workgroup of 1024 threads.
__device__ __forceinline__ uint32_t block_incl_scan(uint32_t x, uint32_t* s_w) {
    const uint32_t lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint32_t inc = x;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)inc, o);
        if ((int)lane >= o) inc += y;
    }
    if (lane == 63) s_w[wid] = inc;
    __syncthreads();
    if (wid == 0) {
        const uint32_t nw = blockDim.x >> 6;
        uint32_t v = lane < nw ? s_w[lane] : 0u;
        uint32_t vi = v;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)vi, o);
            if ((int)lane >= o) vi += y;
        }
        if (lane < nw) s_w[lane] = vi - v;
    }
    __syncthreads();
    const uint32_t r = inc + s_w[wid];
    __syncthreads();
    return r;
}

__global__ void __launch_bounds__(1024) k_scan_tiles(const uint32_t* __restrict__ in, uint32_t n,
                                                     uint32_t* __restrict__ tile_sum) {
    __shared__ uint32_t s_w[16];
    const uint64_t i = (uint64_t)blockIdx.x * 1024 + threadIdx.x;
    const uint32_t x = i < n ? in[i] : 0u;
    const uint32_t inc = block_incl_scan(x, s_w);
    if (threadIdx.x == 1023) tile_sum[blockIdx.x] = inc;
}

__global__ void __launch_bounds__(1024) k_scan_top(uint32_t* __restrict__ tile_sum, uint32_t nt) {
    __shared__ uint32_t s_w[16];
    __shared__ uint32_t s_carry;
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    for (uint32_t base = 0; base < nt; base += 1024) {
        const uint32_t i = base + threadIdx.x;
        const uint32_t x = i < nt ? tile_sum[i] : 0u;
        const uint32_t inc = block_incl_scan(x, s_w);
        const uint32_t carry = s_carry;
        if (i < nt) tile_sum[i] = carry + inc - x;
        __syncthreads();
        if (threadIdx.x == 1023) s_carry = carry + inc;
        __syncthreads();
    }
}

__global__ void __launch_bounds__(1024) k_scan_final(const uint32_t* __restrict__ in, uint32_t n,
                                                     const uint32_t* __restrict__ tile_off,
                                                     uint32_t* __restrict__ out) {
    __shared__ uint32_t s_w[16];
    const uint64_t i = (uint64_t)blockIdx.x * 1024 + threadIdx.x;
    const uint32_t x = i < n ? in[i] : 0u;
    const uint32_t inc = block_incl_scan(x, s_w);
    const uint32_t exc = tile_off[blockIdx.x] + inc - x;
    if (i < n) out[i] = exc;
    if (i == n) out[n] = exc;  // the total (x = 0 there)
}

// The whole scan in one workgroup, 8 counts a lane and step: for few blocks,
// whose scan is one launch's latency instead of three (4.5 us each).
constexpr uint32_t kScanOneMax = 16 * 1024;
__global__ void __launch_bounds__(1024) k_scan_one(const uint32_t* __restrict__ in, uint32_t n,
                                                   uint32_t* __restrict__ out) {
    __shared__ uint32_t s_w[16], s_end;
    uint32_t carry = 0;
    for (uint32_t base = 0; base <= n; base += 8192) {
        const uint32_t i = base + threadIdx.x * 8;
        uint32_t x[8], sum = 0;
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) {
            x[k] = i + k < n ? in[i + k] : 0u;
            sum += x[k];
        }
        const uint32_t inc = block_incl_scan(sum, s_w);  // ends with a barrier
        if (threadIdx.x == 1023) s_end = inc;
        uint32_t at = carry + inc - sum;
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) {
            if (i + k <= n) out[i + k] = at;
            at += x[k];
        }
        __syncthreads();
        carry += s_end;
    }
}

// Group the directory entries by block: segs[seg_off[b] ..] = (first slot,
// count).  Consumes seg_count back to zero.
__global__ void k_fill(PartWs w) {
    if ((w.gate && !*glob(w.gate)) || (w.only_aside && !*glob(w.farcount + 2))) return;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < w.n_chunks * kWin;
         q += stride) {
        const uint64_t c = q / kWin;
        const uint32_t e = (uint32_t)(q % kWin);
        if (e >= w.nd[c]) continue;
        const uint4 d = w.dir[q];
        const uint32_t pos = w.seg_off[d.x] + atomicSub(w.seg_count + d.x, 1u) - 1u;
        w.segs[pos] = make_uint2(d.y, d.z);
    }
}

// Stage 2.  Persistent workgroups take their XCD's blocks in turn (stage2_run).
// A block's segment descriptors (first slot, 16-byte groups) sit in LDS,
// double-buffered: while a block's records are accumulated, the next block's
// descriptors and the segment range of the one after it are in flight.
// Each wave walks its segments (w, w + 8, ...) as one stream of 16-byte groups,
// kRecUnroll loads in flight per lane across segment ends.  The accumulators
// are cleared once and then by the write-out that reads them.
struct Stage2Shared {
    unsigned long long b[4 * kBlockBins];
    uint32_t c[4 * kBlockBins];
    uint32_t start[2][kSegMax];  // first slot (a multiple of 4)
    uint32_t nvec[2][kSegMax];   // 16-byte groups
    uint32_t nseg[2];            // described segments
    uint32_t s0[2], s1[2];       // the block's whole segment range
};

// Where a block's bins go.
struct BlockOut {
    unsigned long long* count;
    unsigned long long* hbytes;
    uint32_t n_bins;
    uint32_t blk;  // the block's index in its stream
    int accumulate;
};

__device__ __forceinline__ void add_record(Stage2Shared& sh, uint32_t r) {
    if (r == 0xFFFFFFFFu) return;  // padding
    const uint32_t key = r >> 20;  // label * kBlockBins + offset
    if (!((r >> 19) & 1u)) {
        atomicAdd(&sh.c[key], 1u);
        atomicAdd(&sh.b[key], (unsigned long long)(r & 0x7FFFFu));
    } else {
        const uint32_t q = (r >> 17) & 3u;
        if (q == 0) atomicAdd(&sh.c[key], 1u);
        atomicAdd(&sh.b[key], (unsigned long long)(r & 0x1FFFFu) << (17 * q));
    }
}

// Accumulate the segments described in buffer d.
__device__ __forceinline__ void stage2_segments(const PartWs& w, Stage2Shared& sh, uint32_t d) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    constexpr uint32_t kWaves = kStage2Block / 64;
    const uint32_t nseg = sh.nseg[d];
    uint32_t j = wave, o = 0;  // the wave's cursor: segment, group offset (wave-uniform)
    while (j < nseg) {
        uint4 r4[kRecUnroll];
#pragma unroll
        for (int u = 0; u < kRecUnroll; ++u) {
            r4[u] = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
            if (j < nseg) {
                const uint32_t nv = sh.nvec[d][j];
                if (o + lane < nv)
                    r4[u] = reinterpret_cast<const uint4*>(w.rec + sh.start[d][j])[o + lane];
                o += 64;
                if (o >= nv) {
                    o = 0;
                    j += kWaves;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kRecUnroll; ++u) {
            add_record(sh, r4[u].x);
            add_record(sh, r4[u].y);
            add_record(sh, r4[u].z);
            add_record(sh, r4[u].w);
        }
    }
}

// Descriptors of segments [s, s + n) of the current block into buffer d
// (n <= kSegMax), by the whole workgroup.
__device__ __forceinline__ void stage2_describe(const PartWs& w, Stage2Shared& sh, uint32_t d,
                                                uint32_t s, uint32_t n) {
    for (uint32_t k = threadIdx.x; k < n; k += kStage2Block) {
        const uint2 sg = w.segs[s + k];
        sh.start[d][k] = sg.x;
        sh.nvec[d][k] = sg.y >> 2;
    }
    if (threadIdx.x == 0) sh.nseg[d] = n;
}

// Bin pairs are written with non-temporal 16-byte stores: the histogram is
// written once and not read back by this pass.
__device__ __forceinline__ void store_pair(unsigned long long* q, unsigned long long x,
                                           unsigned long long y) {
    __builtin_nontemporal_store(u64x2_t{x, y}, glob(reinterpret_cast<u64x2_t*>(q)));
}

// Bins from an output row's start to its first 128-byte line boundary.  Blocks
// start at multiples of kBlockBins bins (8 KB), so a row's skew is the same in
// every block.
__device__ __forceinline__ uint32_t line_skew(const unsigned long long* row) {
    return (uint32_t)(((128u - ((uintptr_t)row & 127u)) & 127u) >> 3);
}

// Write the block's bins and clear the accumulators it read.  Two consecutive
// bins per lane with 16-byte stores when the label rows are 16-byte aligned
// (n_bins even), else one.  Within every row the lanes start at the row's
// first 128-byte line boundary inside the block and wrap around to the bins
// before it, so each wave store covers whole lines and only the two lines a
// block shares with its neighbours are written in part.  On rows that are not
// line-aligned (n_bins * 8 not a multiple of 128, or an offset buffer) wave
// stores that straddle lines cost about a fifth of the write rate.  A block
// without records (empty) writes zeros without touching the accumulators,
// which are already clear.
__device__ __forceinline__ void stage2_write(Stage2Shared& sh, const BlockOut& t, bool empty) {
    const uint64_t b0 = (uint64_t)t.blk * kBlockBins;
    const bool pairs =
        (t.n_bins & 1u) == 0 && (((uintptr_t)t.count | (uintptr_t)t.hbytes) & 15u) == 0;
    if (pairs) {
        const bool zeros = empty && !t.accumulate;
        for (uint32_t k = threadIdx.x; k < 2 * kBlockBins; k += kStage2Block) {
            const uint32_t lab = k / (kBlockBins / 2), j = k % (kBlockBins / 2);
            const uint64_t row = (uint64_t)lab * t.n_bins;
            // skews are even here: the rows are 16-byte aligned
            const uint32_t oc = (line_skew(t.count + row) + 2 * j) & (kBlockBins - 1);
            const uint32_t ob = (line_skew(t.hbytes + row) + 2 * j) & (kBlockBins - 1);
            const uint32_t ec = lab * kBlockBins + oc, eb = lab * kBlockBins + ob;
            ulonglong2 c = make_ulonglong2(0ull, 0ull), b = make_ulonglong2(0ull, 0ull);
            if (!zeros) {
                c = make_ulonglong2(sh.c[ec], sh.c[ec + 1]);
                b = make_ulonglong2(sh.b[eb], sh.b[eb + 1]);
                sh.c[ec] = 0;
                sh.c[ec + 1] = 0;
                sh.b[eb] = 0;
                sh.b[eb + 1] = 0;
            }
            // n_bins even: bin + 1 is inside whenever bin is
            if (b0 + oc < t.n_bins) {
                unsigned long long* q = t.count + row + b0 + oc;
                if (t.accumulate) {
                    const ulonglong2 o = *reinterpret_cast<const ulonglong2*>(q);
                    c.x += o.x;
                    c.y += o.y;
                }
                store_pair(q, c.x, c.y);
            }
            if (b0 + ob < t.n_bins) {
                unsigned long long* q = t.hbytes + row + b0 + ob;
                if (t.accumulate) {
                    const ulonglong2 o = *reinterpret_cast<const ulonglong2*>(q);
                    b.x += o.x;
                    b.y += o.y;
                }
                store_pair(q, b.x, b.y);
            }
        }
    } else {
        for (uint32_t k = threadIdx.x; k < 4 * kBlockBins; k += kStage2Block) {
            const uint32_t lab = k / kBlockBins, j = k % kBlockBins;
            const uint64_t row = (uint64_t)lab * t.n_bins;
            const uint32_t oc = (line_skew(t.count + row) + j) & (kBlockBins - 1);
            const uint32_t ob = (line_skew(t.hbytes + row) + j) & (kBlockBins - 1);
            unsigned long long c = sh.c[lab * kBlockBins + oc], b = sh.b[lab * kBlockBins + ob];
            sh.c[lab * kBlockBins + oc] = 0;
            sh.b[lab * kBlockBins + ob] = 0;
            if (b0 + oc < t.n_bins) {
                unsigned long long* q = t.count + row + b0 + oc;
                *q = t.accumulate ? *q + c : c;
            }
            if (b0 + ob < t.n_bins) {
                unsigned long long* q = t.hbytes + row + b0 + ob;
                *q = t.accumulate ? *q + b : b;
            }
        }
    }
}

// The persistent block loop; out(g) names where block g's bins go.  Runs of
// `run` consecutive blocks are dealt round-robin over the XCDs (workgroup w
// runs on XCD w % kXcds), and an XCD's S workgroups take its blocks in turn.
// With runs of kStage2Run, neighbouring blocks are written at about the same
// time through the same L2, so a 128-byte line that two blocks share (rows
// whose length is not a multiple of 16 bins) is completed there rather than
// written to HBM in two parts, while every XCD still gets a share of every
// part of the histogram.  On 64 uneven streams the batch's stage 2 took
// 5.33-5.35 ms this way, 5.68-5.72 ms with runs of one block and 5.47-5.48 ms
// with one contiguous range per XCD (which also slowed the day cut into 24
// hourly streams, whose busy hours then fell on a few XCDs: 11.33 -> up to
// 11.83 ms).  Where every row starts on a line, runs of one block are faster
// (the 1e8-session day: 1.19 against 1.23 ms).
template <class Out>
__device__ __forceinline__ void stage2_run(const PartWs& w, Stage2Shared& sh, const Out& out,
                                           uint32_t run) {
    const uint32_t tid = threadIdx.x;
    const uint32_t G = gridDim.x, nb = w.n_blocks;
    const uint32_t X = G < (uint32_t)kXcds ? G : (uint32_t)kXcds;  // XCDs with workgroups
    const uint32_t xcd = blockIdx.x % kXcds, lid = blockIdx.x / kXcds;
    const uint32_t per = G / kXcds, rem = G % kXcds;
    const uint32_t S = per + (xcd < rem ? 1u : 0u);  // workgroups on this XCD
    // the XCD's t-th block (increasing in t; nb once past the last block)
    auto blk = [&](uint32_t t) -> uint32_t {
        const uint64_t b = ((uint64_t)(t / run) * X + xcd) * run + t % run;
        return b < nb ? (uint32_t)b : nb;
    };
    uint32_t t = lid;
    uint32_t g = blk(t);
    if (g >= nb) return;
    for (uint32_t k = tid; k < 4 * kBlockBins; k += kStage2Block) {
        sh.b[k] = 0;
        sh.c[k] = 0;
    }
    {
        const uint32_t s0 = w.seg_off[g], s1 = w.seg_off[g + 1];
        stage2_describe(w, sh, 0, s0, min(s1 - s0, (uint32_t)kSegMax));
        if (tid == 0) {
            sh.s0[0] = s0;
            sh.s1[0] = s1;
        }
    }
    uint32_t gn = blk(t + S);  // next block, and its segment range
    uint32_t n0 = 0, n1 = 0;
    if (gn < nb) {
        n0 = w.seg_off[gn];
        n1 = w.seg_off[gn + 1];
    }
    BlockOut cur = out(g);  // where the current block's bins go (found one block ahead)
    for (uint32_t d = 0; g < nb; t += S, g = gn, gn = blk(t + S), d ^= 1u) {
        __syncthreads();  // descriptors of g in buffer d, accumulators clear
        // in flight during this block: the next block's descriptors and the
        // segment range of the block after it
        const uint32_t nn = gn < nb ? min(n1 - n0, (uint32_t)kSegMax) : 0u;
        uint2 nsg = make_uint2(0u, 0u);
        if (tid < nn) nsg = w.segs[n0 + tid];
        const uint32_t gnn = blk(t + 2 * S);
        uint32_t m0 = 0, m1 = 0;
        if (gnn < nb) {
            m0 = w.seg_off[gnn];
            m1 = w.seg_off[gnn + 1];
        }
        const BlockOut nxt = gn < nb ? out(gn) : cur;  // its lookup overlaps this block
        stage2_segments(w, sh, d);
        // blocks with more than kSegMax segments (unsorted input): further
        // batches through the same buffer
        const uint32_t s0 = sh.s0[d], s1 = sh.s1[d];
        for (uint32_t sb = s0 + kSegMax; sb < s1; sb += kSegMax) {
            __syncthreads();
            stage2_describe(w, sh, d, sb, min(s1 - sb, (uint32_t)kSegMax));
            __syncthreads();
            stage2_segments(w, sh, d);
        }
        __syncthreads();  // accumulation complete
        stage2_write(sh, cur, s0 == s1);
        if (gn < nb) {
            const uint32_t e = d ^ 1u;  // last read before this block's first barrier
            if (tid < nn) {
                sh.start[e][tid] = nsg.x;
                sh.nvec[e][tid] = nsg.y >> 2;
            }
            if (tid == 0) {
                sh.nseg[e] = nn;
                sh.s0[e] = n0;
                sh.s1[e] = n1;
            }
        }
        n0 = m0;
        n1 = m1;
        cur = nxt;
    }
}

struct PlainOut {
    unsigned long long* count;
    unsigned long long* hbytes;
    uint32_t n_bins;
    int accumulate;
    __device__ BlockOut operator()(uint32_t g) const {
        return BlockOut{count, hbytes, n_bins, g, accumulate};
    }
};

__global__ void __launch_bounds__(kStage2Block) k_stage2(PartWs w, unsigned long long* count,
                                                        unsigned long long* hbytes, uint32_t n_bins,
                                                        int accumulate) {
    __shared__ Stage2Shared sh;
    if (w.gate && !*glob(w.gate)) return;
    const bool lines = (n_bins & 15u) == 0 && (((uintptr_t)count | (uintptr_t)hbytes) & 127u) == 0;
    stage2_run(w, sh, PlainOut{count, hbytes, n_bins, accumulate}, lines ? 1u : kStage2Run);
}

// A block's accumulators cleared, and added to the output with device atomics
// (both by the whole workgroup).
__device__ __forceinline__ void block_clear(Stage2Shared& sh) {
    for (uint32_t k = threadIdx.x; k < 4 * kBlockBins; k += kStage2Block) {
        sh.b[k] = 0;
        sh.c[k] = 0;
    }
}
__device__ __forceinline__ void block_add(const Stage2Shared& sh, unsigned long long* count,
                                          unsigned long long* hbytes, uint32_t n_bins, uint32_t blk) {
    for (uint32_t k = threadIdx.x; k < 4 * kBlockBins; k += kStage2Block) {
        if (!sh.c[k]) continue;
        const uint64_t x = (uint64_t)(k / kBlockBins) * n_bins + blk * kBlockBins + k % kBlockBins;
        __hip_atomic_fetch_add(count + x, (unsigned long long)sh.c[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(hbytes + x, sh.b[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The records of k_local's runs out of order: a workgroup adds up those of one
// block and a slice of the steps in LDS and then, with device atomics, to the
// output.  Slices, because a block's records are as many as its share of all
// sessions while the blocks are few.
__global__ void __launch_bounds__(kStage2Block) k_deferred(PassParams p, uint32_t* aside, uint32_t slices) {
    __shared__ Stage2Shared sh;
    const DeferWs w = defer_at(aside, p.n, p.n_bins);
    if (*glob(w.any) == 0) return;
    const uint32_t tid = threadIdx.x, blk = blockIdx.x / slices, slice = blockIdx.x - blk * slices;
    const uint32_t t0 = (uint32_t)((uint64_t)w.steps * slice / slices),
                   t1 = (uint32_t)((uint64_t)w.steps * (slice + 1) / slices);
    block_clear(sh);
    PartWs recs{};
    recs.rec = w.rec;
    for (uint32_t t = t0; t < t1; t += kSegMax) {
        const uint32_t n = min(t1 - t, (uint32_t)kSegMax);
        for (uint32_t k = tid; k < n; k += kStage2Block) {
            const uint32_t g = *glob(w.on + t + k) ? *glob(w.dir + (uint64_t)blk * w.steps + t + k) : 0u;
            sh.start[0][k] = (t + k) * kDeferSlots + (g & 0xFFFFu);
            sh.nvec[0][k] = g >> 18;
        }
        if (tid == 0) sh.nseg[0] = n;
        __syncthreads();
        stage2_segments(recs, sh, 0);
        __syncthreads();
    }
    block_add(sh, p.count, p.hbytes, p.n_bins, blk);
}

__global__ void k_zero(unsigned long long* __restrict__ p, uint64_t n) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t head = ((uintptr_t)p & 15) ? 1 : 0;  // p is 8-byte aligned
    if (head && i == 0) p[0] = 0;
    ulonglong2* q = reinterpret_cast<ulonglong2*>(p + head);
    const uint64_t n2 = (n - head) / 2;
    for (uint64_t k = i; k < n2; k += stride) q[k] = make_ulonglong2(0, 0);
    if (i == 0 && ((n - head) & 1)) p[n - 1] = 0;
}

// *gate = 1 (the local reduce does not run) when more than an eighth of 64
// groups of 64 consecutive sessions, evenly spaced, spread over more than
// `spread` bins.  One workgroup of 1,024 lanes, four groups a wave.
__global__ void __launch_bounds__(kMaxBlock) k_local_probe(PassParams p, uint32_t spread,
                                                           uint32_t* gate) {
    __shared__ uint32_t s_wide;
    if (threadIdx.x == 0) s_wide = 0;
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint32_t ts[4];
    bool has[4];
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        const uint64_t i = (p.n >> 6) * (4 * wave + k) + lane;
        has[k] = i < p.n;
        ts[k] = has[k] ? *glob(p.ts + i) : 0u;
    }
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        uint32_t bin;
        const bool in = in_window(p, ts[k], bin) && has[k];
        const uint32_t lo = wave_min(in ? bin : 0xFFFFFFFFu);
        const uint32_t hi = ~wave_min(in ? ~bin : 0xFFFFFFFFu);
        if (lane == 0 && lo <= hi && hi - lo > spread) atomicAdd(&s_wide, 1u);
    }
    __syncthreads();
    if (threadIdx.x == 0) *glob(gate) = s_wide > 8u ? 1u : 0u;
}

// Up to four arrays of 8-byte words cleared in one launch; the first two only
// when the gate (or no gate) says that the local reduce runs.
struct ClearArgs {
    unsigned long long* p[4];
    uint64_t n[4];
    const uint32_t* gate;
};

__global__ void __launch_bounds__(256) k_clear(ClearArgs c) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool local = !c.gate || *glob(c.gate) == 0;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        if (c.n[a] == 0 || (a < 2 && !local)) continue;
        const uint64_t head = ((uintptr_t)c.p[a] & 15) ? 1 : 0;  // 8-byte aligned
        u64x2_t* q = reinterpret_cast<u64x2_t*>(c.p[a] + head);
        const uint64_t n2 = (c.n[a] - head) / 2;
        for (uint64_t k = i; k < n2; k += stride) *glob(q + k) = u64x2_t{0ull, 0ull};
        if (i == 0 && head) *glob(c.p[a]) = 0;
        if (i == 0 && ((c.n[a] - head) & 1)) *glob(c.p[a] + c.n[a] - 1) = 0;
    }
}

// ---------------------------------------------------------------------------
// Batched form: many independent streams in one persistent launch.
//
// The paper's coordinated batch processing feeds uneven chunks through a work
// queue so that every worker stays busy (sections "Coordinated Batch
// Processing", "Work Queue", "TASK DECOMPOSITION").  Here the queue is a
// device counter over (stream, chunk range) items that the persistent
// workgroups pull until it is exhausted; a workgroup restages the table in
// LDS only when the stream changes.  Partitioned streams share one workspace
// (chunk and block index spaces concatenated), so one scan, one fill, one
// stage-2 launch and one far pass serve all of them.  Streams of coarse bins
// take the local reduce instead, an item being a run: their records made a few
// blocks very long, which stage 2 ended on, and their private histograms held a
// CU to one workgroup.  64 streams (3e8 sessions, a third in 1-s bins): stage 1
// 3.20 -> 1.78 ms, stage 2 5.72 -> 3.96 ms, the whole batch 9.27 -> 5.7 to 6.0 ms.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t uniform_u32(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

// Which items of the spare streams are out of order (item.w = 1): as a run of
// k_local, an item is when more than an eighth of 32 of its sessions, evenly spaced,
// lie outside the window that its first 32 sessions place.  Half a wave per item.
// (Asked inside stage 1 it cost all items 3 % there, by registers.)
__global__ void __launch_bounds__(256) k_batch_order(BatchArgs a, uint4* items, PartWs w) {
    const uint32_t it = (blockIdx.x * 256 + threadIdx.x) / 32, l = threadIdx.x & 31u;
    const bool half = (threadIdx.x & 32u) != 0;
    uint32_t first = 0xFFFFFFFFu, bin = 0, bins = 0;
    bool counts = false, spare = false;
    if (it < a.n_items) {
        const uint4 item = items[it];
        const BatchStreamDev& bs = a.streams[item.x];
        spare = bs.spare != 0;
        if (spare) {
            bins = bs.local_bins;
            const uint64_t i0 = (uint64_t)item.y * kChunk, i1 = min(bs.p.n, (uint64_t)item.z * kChunk);
            const uint32_t t0 = *glob(bs.p.ts + min(i0 + l, i1 - 1)), t1 = *glob(bs.p.ts + i0 + (i1 - i0) * l / 32);
            uint32_t b;
            if (in_window(bs.p, t0, b)) first = b;
            counts = in_window(bs.p, t1, bin);
        }
    }
#pragma unroll
    for (int o = 16; o; o >>= 1) first = min(first, (uint32_t)__shfl_xor((int)first, o));
    const uint32_t w0 = first != 0xFFFFFFFFu && first > bins / 16u ? first - bins / 16u : 0u;
    const uint32_t in = (uint32_t)(__ballot(counts) >> (half ? 32 : 0));
    const uint32_t miss = (uint32_t)(__ballot(counts && bin - w0 >= bins) >> (half ? 32 : 0));
    if (it < a.n_items && l == 0) {
        const bool aside = spare && (uint32_t)__popc(miss) * 8u > (uint32_t)__popc(in);
        *glob(&items[it].w) = aside ? 1u : 0u;
        if (aside) *glob(w.farcount + 2) = 1u;
    }
}

template <uint32_t KIND>
__device__ __forceinline__ void batch_stage1(const BatchArgs& a, const PartWs& w) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    __shared__ Stage1Shared sh[2];
    __shared__ uint4 srec[kChunkSlots / 4];
    __shared__ uint32_t s_item;
    __shared__ BatchStreamDev s_bs;  // the current stream's descriptor
    __shared__ uint32_t s_min[kStage1Block / 64];
    const uint32_t tid = threadIdx.x;
    uint32_t staged = 0xFFFFFFFFu;
    LdsView v{};
    uint32_t used = 0;
    uint32_t iter = 0;
    // the local streams' window, then the table
    unsigned long long* win = reinterpret_cast<unsigned long long*>(lds);
    for (uint32_t k = tid; k < a.win_words; k += blockDim.x) win[k] = 0;
    for (;;) {
        if (tid == 0) s_item = atomicAdd(a.counter, 1u);
        __syncthreads();
        const uint32_t it = uniform_u32(s_item);
        if (it >= a.n_items) break;
        const uint4 item = a.items[it];
        const uint32_t si = uniform_u32(item.x);
        if (si != staged) {
            // descriptor to LDS (read there by every lane, never from global
            // memory inside the session loop), then the table
            constexpr uint32_t kWords = sizeof(BatchStreamDev) / 4;
            const uint32_t* src = reinterpret_cast<const uint32_t*>(a.streams + si);
            uint32_t* dst = reinterpret_cast<uint32_t*>(&s_bs);
            for (uint32_t k = tid; k < kWords; k += blockDim.x) dst[k] = src[k];
            __syncthreads();
            v = stage_lds<KIND>(s_bs.p.t, lds + 2 * a.win_words, &used);  // ends with a barrier
            staged = si;
        }
        // the descriptor in scalar registers for the item: read from LDS after
        // every barrier it would cost an LDS round trip per use
        BatchStreamDev bs;
        {
            const uint32_t* src = reinterpret_cast<const uint32_t*>(&s_bs);
            uint32_t* dst = reinterpret_cast<uint32_t*>(&bs);
#pragma unroll
            for (uint32_t k = 0; k < sizeof(BatchStreamDev) / 4; ++k) dst[k] = uniform_u32(src[k]);
        }
        const PassParams& p = bs.p;
        Dropped d{};
        if (bs.local_bins && uniform_u32(item.w) == 0) {  // (k_batch_order: 1 for an item out of order)
            LocalWin w{win, bs.local_bins, bs.reps, 0u};
            const bool vec = bs.vec != 0;
            auto full = [&](uint64_t c) { return vec && (c + 1) * kChunk <= p.n; };
            const uint32_t rep = tid & ((1u << bs.reps) - 1u);
            Raw4 cur{}, nxt{};
            uint64_t c = item.y;
            if (c < item.z && full(c)) load4<KIND>(p, c * kChunk + 4ull * tid, cur);
            if (bs.local_bins < p.n_bins)
                w.w0 = local_place(local_first(p, c * kChunk + 4ull * tid, cur, full(c)), w.bins, s_min);
            for (; c < item.z; ++c) {
                if (c + 1 < item.z && full(c + 1)) load4<KIND>(p, (c + 1) * kChunk + 4ull * tid, nxt);
                local_add4<KIND>(p, v, w, rep, c * kChunk + 4ull * tid, cur, full(c), d);
                cur = nxt;
            }
            __syncthreads();
            local_flush(p, w);  // cleared before the next item's first barrier
        } else {
            const bool vec = bs.vec != 0;
            auto full = [&](uint64_t c) { return vec && (c + 1) * kChunk <= p.n; };
            Raw4 cur{}, nxt{};
            uint64_t c = item.y;
            if (c < item.z && full(c)) load4<KIND>(p, c * kChunk + (uint64_t)tid * 4, cur);
            for (; c < item.z; ++c) {
                if (c + 1 < item.z && full(c + 1)) load4<KIND>(p, (c + 1) * kChunk + (uint64_t)tid * 4, nxt);
                stage1_chunk<KIND>(p, w, v, sh[iter++ & 1u], srec, c, bs.chunk0 + c, bs.block0, cur,
                                   full(c), d);
                cur = nxt;
            }
        }
        d.flush(p.dropped);
    }
}

// Block g of the shared workspace belongs to the last stream whose first
// block is <= g (streams without blocks share their base with the next one).
struct BatchOut {
    const BatchArgs* a;
    __device__ BlockOut operator()(uint32_t gb) const {
        uint32_t lo = 0, n = a->n_streams;
        while (n > 1) {
            const uint32_t half = n >> 1;
            lo = a->block_base[lo + half] <= gb ? lo + half : lo;
            n -= half;
        }
        while (lo + 1 < a->n_streams && a->block_base[lo + 1] <= gb) ++lo;
        const BatchStreamDev& bs = a->streams[lo];
        return BlockOut{bs.p.count, bs.p.hbytes, bs.p.n_bins, gb - bs.block0, 0};
    }
};

__global__ void __launch_bounds__(kStage2Block) k_batch_stage2(BatchArgs a, PartWs w) {
    __shared__ Stage2Shared sh;
    stage2_run(w, sh, BatchOut{&a}, kStage2Run);
}

// The blocks (stream, block) of the local streams whose items out of order became
// records: added to what their other items put into the output.
__global__ void __launch_bounds__(kStage2Block) k_batch_aside(BatchArgs a, PartWs w, const uint2* blocks,
                                                              uint32_t slices) {
    __shared__ Stage2Shared sh;
    if (*glob(w.farcount + 2) == 0) return;
    const uint32_t slice = blockIdx.x % slices;
    const uint2 id = blocks[blockIdx.x / slices];
    const BatchStreamDev& bs = a.streams[id.x];
    const uint32_t s0 = w.seg_off[bs.block0 + id.y], n = w.seg_off[bs.block0 + id.y + 1] - s0;
    const uint32_t t0 = s0 + (uint32_t)((uint64_t)n * slice / slices),
                   t1 = s0 + (uint32_t)((uint64_t)n * (slice + 1) / slices);
    if (t0 == t1) return;
    block_clear(sh);
    for (uint32_t t = t0; t < t1; t += kSegMax) {
        stage2_describe(w, sh, 0, t, min(t1 - t, (uint32_t)kSegMax));
        __syncthreads();
        stage2_segments(w, sh, 0);
        __syncthreads();
    }
    block_add(sh, bs.p.count, bs.p.hbytes, bs.p.n_bins, id.y);
}


// In/out-index lookups fit 128 VGPRs (4 waves per SIMD, two workgroups per CU);
// the interval kinds keep their registers rather than spill.
template <uint32_t KIND>
__global__ void __launch_bounds__(kStage1Block) k_batch_stage1(BatchArgs a, PartWs w) {
    batch_stage1<KIND>(a, w);
}
template <uint32_t KIND>
__global__ void __launch_bounds__(kStage1Block, 4) k_batch_stage1_o4(BatchArgs a, PartWs w) {
    batch_stage1<KIND>(a, w);
}

template <uint32_t KIND>
__global__ void __launch_bounds__(kMaxBlock) k_batch_far(BatchArgs a, PartWs w) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    uint32_t staged = 0xFFFFFFFFu;
    LdsView v{};
    uint32_t used = 0;
    const uint32_t nfar = *w.farcount;
    for (uint32_t q = blockIdx.x; q < nfar; q += gridDim.x) {
        const uint64_t g = w.farlist[q];
        uint32_t lo = 0, n = a.n_streams;
        while (n > 1) {
            const uint32_t half = n >> 1;
            lo = a.chunk_base[lo + half] <= g ? lo + half : lo;
            n -= half;
        }
        while (lo + 1 < a.n_streams && a.chunk_base[lo + 1] <= g) ++lo;
        const uint32_t si = uniform_u32(lo);
        const BatchStreamDev& bs = a.streams[si];
        if (bs.p.t.kind != KIND) continue;  // another kind group's chunk
        PassParams p = bs.p;
        p.label_out = nullptr;
        p.src_inst = nullptr;
        p.dst_inst = nullptr;
        p.dropped = nullptr;
        if (si != staged) {
            __syncthreads();
            v = stage_lds<KIND>(p.t, lds, &used);
            staged = si;
        }
        const uint64_t c = g - bs.chunk0;
        Dropped d{};
        for (uint32_t s = threadIdx.x; s < kChunk; s += blockDim.x) {
            const uint64_t i = c * kChunk + s;
            if (i < p.n && ((w.farbits[g * (kChunk / 32) + s / 32] >> (s & 31)) & 1u))
                one_session<KIND, H_ATOMIC>(p, v, i, d);
        }
    }
}

// Batched lookup pass: streams whose lookups walk global memory store their
// labels first, as the single-stream path does, and stage 1 reads them (one
// byte per session) instead of stalling its barriers on the lookups.  Work
// items as in batch stage 1; a workgroup restages the table only when the
// stream changes; the next four sessions' addresses are loaded before the
// current ones are looked up.
template <uint32_t KIND>
__global__ void __launch_bounds__(kMaxBlock) k_batch_lookup(BatchArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    __shared__ uint32_t s_item;
    __shared__ BatchStreamDev s_bs;
    const uint32_t tid = threadIdx.x;
    uint32_t staged = 0xFFFFFFFFu;
    LdsView v{};
    uint32_t used = 0;
    for (;;) {
        __syncthreads();  // every lane is done with the previous item
        if (tid == 0) s_item = atomicAdd(a.counter, 1u);
        __syncthreads();
        const uint32_t it = uniform_u32(s_item);
        if (it >= a.n_items) break;
        const uint4 item = a.items[it];
        const uint32_t si = uniform_u32(item.x);
        if (si != staged) {
            constexpr uint32_t kWords = sizeof(BatchStreamDev) / 4;
            const uint32_t* src = reinterpret_cast<const uint32_t*>(a.streams + si);
            uint32_t* dst = reinterpret_cast<uint32_t*>(&s_bs);
            for (uint32_t k = tid; k < kWords; k += blockDim.x) dst[k] = src[k];
            __syncthreads();
            v = stage_lds<KIND>(s_bs.p.t, lds, &used);  // ends with a barrier
            // the window PLA's search queue, after the table (a.queue_words
            // per wave when the launch made room for it)
            if constexpr (KIND == KK_PLA)  // window PLAs only (the wider search needs a larger queue)
                v.queue = a.queue_words && s_bs.p.t.pla_window
                              ? (__attribute__((address_space(3))) uint32_t*)(lds + used + (tid >> 6) * a.queue_words)
                              : nullptr;
            staged = si;
        }
        BatchStreamDev bs;
        {
            const uint32_t* src = reinterpret_cast<const uint32_t*>(&s_bs);
            uint32_t* dst = reinterpret_cast<uint32_t*>(&bs);
#pragma unroll
            for (uint32_t k = 0; k < sizeof(BatchStreamDev) / 4; ++k) dst[k] = uniform_u32(src[k]);
        }
        const PassParams& p = bs.p;
        const uint64_t groups = (p.n + 3) / 4;
        const uint64_t g0 = (uint64_t)item.y * (kChunk / 4);
        const uint64_t g1 = min((uint64_t)item.z * (kChunk / 4), groups);
        auto full = [&](uint64_t g) { return bs.vec && g * 4 + 4 <= p.n; };
        uint4 cs = make_uint4(0, 0, 0, 0), cd = cs, ns = cs, nd = cs;
        uint64_t g = g0 + tid;
        if (g < g1 && full(g)) {
            cs = gload4(p.src + g * 4);
            cd = gload4(p.dst + g * 4);
        }
        for (; g < g1; g += blockDim.x) {
            const uint64_t gn = g + blockDim.x;
            if (gn < g1 && full(gn)) {
                ns = gload4(p.src + gn * 4);
                nd = gload4(p.dst + gn * 4);
            }
            if (full(g)) {
                uint32_t lab[4];
                labels4_from<KIND, KIND == KK_PLA ? kQueueWindow : 0>(p, v, g * 4, cs, cd, 0u, lab);
            } else {
                Dropped d{};
                for (uint64_t i = g * 4; i < p.n && i < g * 4 + 4; ++i)
                    one_session<KIND, H_NONE>(p, v, i, d);
            }
            cs = ns;
            cd = nd;
        }
    }
}

__global__ void k_zero_jobs(const ZeroJob* __restrict__ jobs, uint32_t n_jobs) {
    for (uint32_t j = blockIdx.x; j < n_jobs; j += gridDim.x) {
        const ZeroJob z = jobs[j];
        for (uint64_t k = threadIdx.x; k < z.n; k += blockDim.x) z.p[k] = 0;
    }
}

// ---------------------------------------------------------------------------
// Watch-list histograms (sections "AbuseIPDB" and "GRIZZLY STEPPE", Figures
// 8-11): the sessions of listed hosts per time window, in both directions.
// The list is a prefix table whose institution ids are the keys.  Each
// session looks up its source and its destination; a match adds (1, bytes)
// to cell [dir][key][bin] (dir 0: the source matched, 1: the destination),
// or to dropped[dir] outside the window.  Listed sessions are few, so the
// pass is a streaming read of the address columns: the /16 filter in LDS
// rejects most addresses with one LDS read, only addresses in blocks the
// list touches run the interval search, and the timestamps and byte counts
// are loaded only for matches.  Bound by the address read and vector issue:
// searched in every iteration, a wave paid a whole search round (12 steps and
// the matches' loads) for about a dozen addresses, and eight ballots to queue
// them; collected over iterations and queued one per lane and round, 4e8
// sessions with 1,177 hosts take 0.67 ms instead of 0.92 (4.8 TB/s).  Small
// histograms live in LDS per workgroup (merged with atomics at the end);
// larger ones take device-scope atomics directly.
// ---------------------------------------------------------------------------
constexpr int kWatchBlock = 512;
constexpr uint32_t kWatchPrivCells = 4096;  // [2][n_keys][n_bins] cells kept in LDS
constexpr uint32_t kWatchLdsKeys = 8192;    // intervals whose keys are staged in LDS

struct WatchParams {
    PassParams p;       // list table, columns, window; count/hbytes [2][n_keys][n_bins], dropped [2][2]
    uint32_t n_keys;
    uint32_t vec;       // 16-byte loads allowed
    uint32_t lds_keys;  // 1: key + 1 of every interval staged in LDS (m <= kWatchLdsKeys)
    uint32_t pad;
};

// Longest-match row + 1 (0: no match) of each address.
template <uint32_t KIND, int N>
__device__ __forceinline__ void owners(const DevTable& t, const LdsView& v, const uint32_t* a,
                                       uint32_t* code) {
    if constexpr (KIND == KK_SCAN) {
#pragma unroll
        for (int q = 0; q < N; ++q) code[q] = scan_owner(t, v, a[q]);
    } else {
        uint32_t need = 0;
#pragma unroll
        for (int q = 0; q < N; ++q) {
            code[q] = 0;
            const uint32_t st = (v.filter[a[q] >> 20] >> (((a[q] >> 16) & 15u) * 2)) & 3u;
            need |= (st != 0u ? 1u : 0u) << q;
        }
        if (need) {
            uint32_t j[N];
            intervals<KIND, N>(t, v, a, j, need);
#pragma unroll
            for (int q = 0; q < N; ++q)
                if ((need >> q) & 1u) code[q] = *glob(t.owner + j[q]);
        }
    }
}

struct WatchDropped {
    unsigned long long c[2], b[2];
    __device__ __forceinline__ void add(uint32_t dir, uint64_t nbytes) {
        c[dir] += 1;
        b[dir] += nbytes;
    }
    __device__ __forceinline__ void flush(unsigned long long* out) const {
        if (!out) return;
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            if (c[d]) {
                atomicAdd(out + 2 * d, c[d]);
                atomicAdd(out + 2 * d + 1, b[d]);
            }
        }
    }
};

// code: key + 1 when is_key, else the owner row + 1 (its key read from the
// table's inst ids).
template <bool PRIV>
__device__ __forceinline__ void watch_add(const WatchParams& w, uint32_t* hc, unsigned long long* hb,
                                          uint32_t dir, uint32_t code, bool is_key, uint32_t ts,
                                          uint64_t nbytes, WatchDropped& d) {
    uint32_t bin;
    if (!in_window(w.p, ts, bin)) {
        d.add(dir, nbytes);
        return;
    }
    const uint32_t key = is_key ? code - 1 : *glob(w.p.t.inst + (code - 1));
    const uint64_t k = ((uint64_t)dir * w.n_keys + key) * w.p.n_bins + bin;
    if constexpr (PRIV) {
        atomicAdd(hc + k, 1u);
        atomicAdd(hb + k, (unsigned long long)nbytes);
    } else {
        __hip_atomic_fetch_add(w.p.count + k, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(w.p.hbytes + k, (unsigned long long)nbytes, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Addresses that the /16 filter lets through, per wave in LDS: the address and
// where it came from (iteration << 9 | lane << 3 | session << 1 | direction).
// Few are let through (2 % with 1,177 hosts), so they are collected over
// iterations and searched 64 at a time, one per lane; a lane whose address is on
// the list then loads that session's time and byte count and adds it.
constexpr uint32_t kWatchQueue = 128;  // entries of a wave: fewer than 64 kept and 64 added

template <uint32_t KIND, bool PRIV>
__global__ void __launch_bounds__(kWatchBlock) k_watch(WatchParams w) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    uint32_t used = 0;
    const PassParams& p = w.p;
    const LdsView v = stage_lds<KIND>(p.t, lds, &used);
    uint32_t* qa = lds + used + (threadIdx.x >> 6) * (2 * kWatchQueue);  // this wave's queue
    uint32_t* qi = qa + kWatchQueue;
    if constexpr (KIND != KK_SCAN) used += (kWatchBlock / 64) * 2 * kWatchQueue;
    // key + 1 (0: no match) of every interval, when the list is small enough
    uint32_t* lkey = nullptr;
    if constexpr (KIND != KK_SCAN) {
        if (w.lds_keys) {
            lkey = lds + used;
            for (uint32_t j = threadIdx.x; j < p.t.m; j += blockDim.x) {
                const uint32_t o = *glob(p.t.owner + j);
                lkey[j] = o ? *glob(p.t.inst + (o - 1)) + 1u : 0u;
            }
            used += p.t.m;
            __syncthreads();
        }
    }
    uint32_t* hc = nullptr;
    unsigned long long* hb = nullptr;
    const uint32_t cells = 2u * w.n_keys * p.n_bins;  // <= kWatchPrivCells when PRIV
    if constexpr (PRIV) {
        used = (used + 1) & ~1u;
        hb = reinterpret_cast<unsigned long long*>(lds + used);
        hc = lds + used + 2 * cells;
        for (uint32_t k = threadIdx.x; k < cells; k += blockDim.x) {
            hb[k] = 0;
            hc[k] = 0;
        }
        __syncthreads();
    }
    WatchDropped d{};
    const uint64_t groups = (p.n + 3) / 4;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint32_t lane = lane_id();
    const uint64_t g0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, wave_g0 = g0 - lane;
    // the next group's addresses are loaded while this one is looked up
    auto full = [&](uint64_t g) { return w.vec && g * 4 + 4 <= p.n; };
    uint4 cs = make_uint4(0, 0, 0, 0), cd = cs;
    if (full(g0)) {
        cs = gload4_nt(p.src + g0 * 4);
        cd = gload4_nt(p.dst + g0 * 4);
    }
    uint32_t held = 0;  // entries of the wave's queue (wave-uniform)
    // search and add the queue's last 64 entries (or all that are left)
    auto drain = [&]() {
        const uint32_t n = min(held, 64u);
        held -= n;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        if (lane < n) {
            const uint32_t x = qa[held + lane], id = qi[held + lane];
            uint32_t j;
            intervals<KIND == KK_SCAN ? KK_BSEARCH : KIND, 1>(p.t, v, &x, &j, 1u);
            const uint32_t code = lkey ? lkey[j] : *glob(p.t.owner + j);
            if (code) {
                const uint64_t i = (wave_g0 + (id >> 9) * stride + ((id >> 3) & 63u)) * 4 + ((id >> 1) & 3u);
                watch_add<PRIV>(w, hc, hb, id & 1u, code, lkey != nullptr, *glob(p.ts + i), *glob(p.bytes + i), d);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // its slots are written again
    };
    uint32_t it = 0;
    for (uint64_t wg = wave_g0; wg < groups; wg += stride, ++it) {  // wave-uniform
        const uint64_t g = wg + lane, i = g * 4;
        uint4 ns = cs, nd = cd;
        if (full(g + stride)) {
            ns = gload4_nt(p.src + (g + stride) * 4);
            nd = gload4_nt(p.dst + (g + stride) * 4);
        }
        const uint32_t a[8] = {cs.x, cs.y, cs.z, cs.w, cd.x, cd.y, cd.z, cd.w};
        if constexpr (KIND != KK_SCAN) {
            uint32_t need = 0;  // bit q: address q may be on the list
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const uint32_t st = (v.filter[a[q] >> 20] >> (((a[q] >> 16) & 15u) * 2)) & 3u;
                need |= (st != 0u ? 1u : 0u) << q;
            }
            if (!full(g)) need = 0;
            // each lane queues one of its addresses per round
            for (uint64_t m = __ballot(need != 0u); m; m = __ballot(need != 0u)) {
                if (need) {
                    const uint32_t q = (uint32_t)__builtin_ctz(need), at = held + rank_in(m);
                    const uint32_t lo = q & 2u ? (q & 1u ? cs.w : cs.z) : (q & 1u ? cs.y : cs.x);
                    const uint32_t hi = q & 2u ? (q & 1u ? cd.w : cd.z) : (q & 1u ? cd.y : cd.x);
                    qa[at] = q & 4u ? hi : lo;
                    qi[at] = it << 9 | lane << 3 | (q & 3u) << 1 | q >> 2;
                    need &= need - 1u;
                }
                held += (uint32_t)__popcll(m);
                if (held >= 64u) drain();
            }
        } else if (full(g)) {
            uint32_t code[8], any = 0;
            owners<KIND, 8>(p.t, v, a, code);
#pragma unroll
            for (int q = 0; q < 8; ++q) any |= code[q];
            if (any) {
                const uint4 ts = gload4(p.ts + i);
                const ulonglong2 b01 = gload2(p.bytes + i), b23 = gload2(p.bytes + i + 2);
                const uint32_t t4[4] = {ts.x, ts.y, ts.z, ts.w};
                const uint64_t by[4] = {b01.x, b01.y, b23.x, b23.y};
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (code[q]) watch_add<PRIV>(w, hc, hb, q >> 2, code[q], false, t4[q & 3], by[q & 3], d);
            }
        }
        if (!full(g)) {  // the ragged last group, or unaligned columns
            for (uint64_t e = i; e < p.n && e < i + 4; ++e) {
                const uint32_t x[2] = {*glob(p.src + e), *glob(p.dst + e)};
                uint32_t code[2];
                owners<KIND, 2>(p.t, v, x, code);
                if (code[0] | code[1]) {
                    const uint32_t ts = *glob(p.ts + e);
                    const uint64_t by = *glob(p.bytes + e);
                    for (uint32_t dir = 0; dir < 2; ++dir)
                        if (code[dir]) watch_add<PRIV>(w, hc, hb, dir, code[dir], false, ts, by, d);
                }
            }
        }
        cs = ns;
        cd = nd;
    }
    if constexpr (KIND != KK_SCAN)
        while (held) drain();
    d.flush(p.dropped);
    if constexpr (PRIV) {
        __syncthreads();
        for (uint32_t k = threadIdx.x; k < cells; k += blockDim.x) {
            if (hc[k]) {
                __hip_atomic_fetch_add(p.count + k, (unsigned long long)hc[k], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_fetch_add(p.hbytes + k, hb[k], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
using PassFn = void (*)(PassParams, FarList);
using Stage1Fn = void (*)(PassParams, PartWs);

template <uint32_t KIND>
static PassFn pass_fn(int hm, bool vec) {
    if (KIND == KK_INOUT && hm == H_NONE && vec) return k_pass_inout;
    if (hm == H_NONE) return vec ? k_pass<KIND, H_NONE, true> : k_pass<KIND, H_NONE, false>;
    return vec ? k_pass<KIND, H_ATOMIC, true> : k_pass<KIND, H_ATOMIC, false>;
}

static PassFn pick_pass(uint32_t kind, int hm, bool vec) {
    switch (kind) {
        case KK_SCAN: return pass_fn<KK_SCAN>(hm, vec);
        case KK_BSEARCH: return pass_fn<KK_BSEARCH>(hm, vec);
        case KK_TRIE: return pass_fn<KK_TRIE>(hm, vec);
        case KK_PLA: return pass_fn<KK_PLA>(hm, vec);
        case KK_MLP: return pass_fn<KK_MLP>(hm, vec);
        case KK_INOUT: return pass_fn<KK_INOUT>(hm, vec);
        case KK_UNION: return pass_fn<KK_UNION>(hm, vec);
        case KK_LABEL_IN: return pass_fn<KK_LABEL_IN>(hm, vec);
        default: return nullptr;
    }
}

static Stage1Fn pick_stage1(uint32_t kind) {
    switch (kind) {
        case KK_SCAN: return k_stage1<KK_SCAN>;
        case KK_BSEARCH: return k_stage1<KK_BSEARCH>;
        case KK_TRIE: return k_stage1<KK_TRIE>;
        case KK_PLA: return k_stage1<KK_PLA>;
        case KK_MLP: return k_stage1<KK_MLP>;
        case KK_INOUT: return k_stage1<KK_INOUT>;
        case KK_UNION: return k_stage1<KK_UNION>;
        case KK_LABEL_IN: return k_stage1<KK_LABEL_IN>;
        default: return nullptr;
    }
}

uint32_t device_cu_count() {
    static std::mutex mu;
    static std::map<int, uint32_t> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    std::lock_guard<std::mutex> g(mu);
    auto it = cache.find(dev);
    if (it != cache.end()) return it->second;
    hipDeviceProp_t prop;
    uint32_t cus = 256;
    if (hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0)
        cus = (uint32_t)prop.multiProcessorCount;
    cache[dev] = cus;
    return cus;
}

int blocks_per_cu(const void* fn, int block, size_t lds) {
    static std::mutex mu;
    static std::map<std::tuple<const void*, int, size_t, int>, int> cache;
    int dev = 0;
    (void)hipGetDevice(&dev);
    auto key = std::make_tuple(fn, block, lds, dev);
    std::lock_guard<std::mutex> g(mu);
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    if (lds > 64 * 1024)
        (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, block, lds) != hipSuccess || nb < 1)
        nb = 1;
    // The answer divides the 160 KB by the bytes asked for, but LDS is handed
    // out in 1,280-byte granules: five workgroups of 32 KB are reported and
    // four are resident, and a grid for five runs a fifth round of a quarter
    // of its workgroups (0.91 against 0.69 ms for 2e8 addresses).
    hipFuncAttributes at{};
    if (hipFuncGetAttributes(&at, fn) == hipSuccess) {
        const size_t granules = (lds + at.sharedSizeBytes + 1279) / 1280;
        if (granules) nb = std::max(1, std::min(nb, (int)(128 / granules)));
    }
    cache[key] = nb;
    return nb;
}

uint64_t div_magic(uint32_t width) {
    return width >= 2 ? (~0ull) / width + 1 : 0ull;
}

static bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }
static bool aligned4(const void* p) { return ((uintptr_t)p & 3u) == 0; }

// Can the 4-session vector loads/stores be used for these pointers?
bool vector_ok(const PassParams& p, uint32_t kind, bool hist) {
    if (p.pos_out) return aligned16(p.src) && aligned16(p.pos_out);
    bool vec = true;
    if (kind == KK_LABEL_IN) vec = aligned4(p.label_in);
    else vec = aligned16(p.src) && aligned16(p.dst);
    if (p.label_out) vec = vec && aligned4(p.label_out);
    if (p.src_inst) vec = vec && aligned16(p.src_inst);
    if (p.dst_inst) vec = vec && aligned16(p.dst_inst);
    if (hist) vec = vec && aligned16(p.ts) && aligned16(p.bytes);
    return vec;
}

static sinet_status launch_k_pass(const PassParams& p, uint32_t kind, int hm, bool vec,
                                  const FarList& far, hipStream_t s) {
    PassFn fn = pick_pass(kind, hm, vec);
    if (!fn) return fail(SINET_ERR_UNSUPPORTED, "no kernel for this lookup kind");
    size_t lds = (kind == KK_LABEL_IN ? 0 : p.t.lds_bytes) + 8;
    if (lds > 160 * 1024) return fail(SINET_ERR_UNSUPPORTED, "table needs more LDS than a CU has");
    const int block = lds > 40 * 1024 ? 1024 : 256;
    // the lookup pass of the queued kinds queues its searches per wave when
    // the queues fit beside the table (labels only: positions and institution
    // ids take the direct path)
    PassParams q = p;
    q.queue_words = 0;
    // (the binary search over all boundaries in global memory, one leaf, is
    // latency-bound like the PLA and keeps the direct path)
    const bool global_search = kind == KK_BSEARCH && p.t.n_top <= 1;
    const uint32_t qw = kind == KK_PLA && p.t.pla_window ? kPlaQueue : kSearchQueue;
    if (hm == H_NONE && queued_kind(kind) && qw && !global_search && !p.pos_out && !p.src_inst &&
        !p.dst_inst && lds + (size_t)(block / 64) * qw * 4 <= 160 * 1024) {
        q.queue_words = qw;
        lds += (size_t)(block / 64) * qw * 4;
    }
    uint64_t grid = (uint64_t)device_cu_count() * blocks_per_cu((const void*)fn, block, lds);
    if (!far.list) {
        const uint64_t tiles = ((p.n + 3) / 4 + block - 1) / block;
        if (grid > tiles) grid = tiles;
    }
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(block), lds, s, q, far);
    return check_hip(hipGetLastError(), "pass kernel launch");
}

sinet_status launch_pass(const PassParams& p, uint32_t mode, hipStream_t s) {
    if (p.n == 0) return SINET_OK;
    const uint32_t kind = (mode & PASS_LABEL_IN) ? (uint32_t)KK_LABEL_IN : p.t.kind;
    const bool hist = (mode & PASS_HIST) != 0;
    FarList none{};
    return launch_k_pass(p, kind, hist ? H_ATOMIC : H_NONE, vector_ok(p, kind, hist), none, s);
}

sinet_status launch_zero(unsigned long long* p, uint64_t n_words, hipStream_t s) {
    if (n_words == 0) return SINET_OK;
    uint64_t blocks = (n_words / 2 + 255) / 256;
    const uint64_t cap = (uint64_t)device_cu_count() * 8;
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_zero, dim3((unsigned)blocks), dim3(256), 0, s, p, n_words);
    return check_hip(hipGetLastError(), "zero kernel launch");
}

// The histogram's arrays (cells words each; with a gate only if it says so) and
// dropped counters cleared in one launch; dropped may be NULL, cells 0.
static sinet_status launch_clears(const ClearArgs& c, hipStream_t s) {
    const uint64_t most = c.n[0] > c.n[1] ? c.n[0] : c.n[1];
    if (most + c.n[2] + c.n[3] == 0) return SINET_OK;
    uint64_t blocks = (most / 2 + 255) / 256;
    const uint64_t cap = (uint64_t)device_cu_count() * 8;
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_clear, dim3((unsigned)blocks), dim3(256), 0, s, c);
    return check_hip(hipGetLastError(), "clear launch");
}

static sinet_status launch_clear(const PassParams& p, uint64_t cells, hipStream_t s,
                                 const uint32_t* gate = nullptr) {
    return launch_clears({{p.count, p.hbytes, p.dropped}, {cells, cells, p.dropped ? 8ull : 0ull}, gate}, s);
}

// ---- workspace of the partitioned histogram --------------------------------
static size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

// Persistent stage-2 workgroups: as many as fit on the device at once.
static uint32_t stage2_grid(uint32_t n_blocks) {
    static const uint32_t per_cu = (uint32_t)blocks_per_cu((const void*)k_stage2, kStage2Block, 0);
    const uint64_t g = (uint64_t)device_cu_count() * (per_cu ? per_cu : 1u);
    return (uint32_t)(g < n_blocks ? g : n_blocks);
}

size_t part_ws_bytes(uint64_t n, uint32_t n_bins) {
    const uint64_t nc = (n + kChunk - 1) / kChunk;
    const uint64_t nb = (n_bins + kBlockBins - 1) / kBlockBins;
    const uint64_t nt = (nb + 1 + 1023) / 1024;
    return al256(4 * nc * kChunkSlots) + al256(16 * nc * kWin) +
           al256(4 * nc) + al256(4 * nc * (kChunk / 32)) + al256(4 * (nc + 1)) + al256(4 * nb) +
           al256(4 * (nb + 1)) + al256(8 * nc * kWin) + al256(4 * nt) + 256;
}

PartWs part_ws_carve(void* base, uint64_t n, uint32_t n_bins) {
    PartWs w{};
    const uint64_t nc = (n + kChunk - 1) / kChunk;
    const uint64_t nb = (n_bins + kBlockBins - 1) / kBlockBins;
    const uint64_t nt = (nb + 1 + 1023) / 1024;
    char* a = (char*)base;
    size_t o = 0;
    auto take = [&](size_t bytes) { char* r = a + o; o += al256(bytes); return (void*)r; };
    w.rec = (uint32_t*)take(4 * nc * kChunkSlots);
    w.dir = (uint4*)take(16 * nc * kWin);
    w.nd = (uint32_t*)take(4 * nc);
    w.farbits = (uint32_t*)take(4 * nc * (kChunk / 32));
    w.farlist = (uint32_t*)take(4 * (nc + 1));
    w.seg_count = (uint32_t*)take(4 * nb);
    w.seg_off = (uint32_t*)take(4 * (nb + 1));
    w.segs = (uint2*)take(8 * nc * kWin);
    w.scan_tiles = (uint32_t*)take(4 * nt);
    w.farcount = (uint32_t*)take(256);
    w.next_run = w.farcount + 1;
    w.n_chunks = nc;
    w.n_blocks = (uint32_t)nb;
    return w;
}

// Segment index: exclusive scan of the per-block directory counts, then the
// fill that groups directory entries by block.
sinet_status launch_scan_fill(const PartWs& w, hipStream_t s) {
    const uint32_t nb = w.n_blocks;
    const uint32_t ntiles = (nb + 1 + 1023) / 1024;
    if (nb < kScanOneMax) {
        hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(1024), 0, s, w.seg_count, nb, w.seg_off);
    } else {
        hipLaunchKernelGGL(k_scan_tiles, dim3(ntiles), dim3(1024), 0, s, w.seg_count, nb, w.scan_tiles);
        hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, s, w.scan_tiles, ntiles);
        hipLaunchKernelGGL(k_scan_final, dim3(ntiles), dim3(1024), 0, s, w.seg_count, nb, w.scan_tiles,
                           w.seg_off);
    }
    uint64_t fb = (w.n_chunks * kWin + 255) / 256;
    const uint64_t cap = (uint64_t)device_cu_count() * 16;
    if (fb > cap) fb = cap;
    if (fb < 1) fb = 1;
    hipLaunchKernelGGL(k_fill, dim3((unsigned)fb), dim3(256), 0, s, w);
    return check_hip(hipGetLastError(), "segment index launch");
}

// ---- phase timing ------------------------------------------------------------
// While enabled, every phase of run_hist is bracketed by two events recorded on
// the launch stream; they are read (and destroyed) by timing_read.
namespace {
struct Mark {
    int phase;
    hipEvent_t a, b;
};
std::mutex g_tm_mu;
bool g_tm_on = false;
std::vector<Mark> g_tm_marks;
uint64_t g_tm_calls = 0;
uint64_t g_tm_window = 0;

class PhaseScope {
   public:
    PhaseScope(int phase, hipStream_t s, bool enabled = true) : phase_(phase), s_(s) {
        if (!enabled) return;
        {
            std::lock_guard<std::mutex> g(g_tm_mu);
            if (!g_tm_on) return;
        }
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) return;
        if (hipEventCreate(&a_) != hipSuccess) return;
        if (hipEventCreate(&b_) != hipSuccess) {
            (void)hipEventDestroy(a_);
            return;
        }
        on_ = hipEventRecord(a_, s) == hipSuccess;
        if (!on_) {
            (void)hipEventDestroy(a_);
            (void)hipEventDestroy(b_);
        }
    }
    ~PhaseScope() {
        if (!on_) return;
        (void)hipEventRecord(b_, s_);
        std::lock_guard<std::mutex> g(g_tm_mu);
        g_tm_marks.push_back(Mark{phase_, a_, b_});
    }
    PhaseScope(const PhaseScope&) = delete;
    PhaseScope& operator=(const PhaseScope&) = delete;

   private:
    int phase_;
    hipStream_t s_;
    hipEvent_t a_{}, b_{};
    bool on_ = false;
};

void count_timed_call() {
    std::lock_guard<std::mutex> g(g_tm_mu);
    if (g_tm_on) ++g_tm_calls;
}

void count_window_call() {
    std::lock_guard<std::mutex> g(g_tm_mu);
    if (g_tm_on) ++g_tm_window;
}

void drop_marks_locked() {
    for (const Mark& m : g_tm_marks) {
        (void)hipEventDestroy(m.a);
        (void)hipEventDestroy(m.b);
    }
    g_tm_marks.clear();
    g_tm_calls = 0;
    g_tm_window = 0;
}
}  // namespace

sinet_status timing_enable(int on) {
    std::lock_guard<std::mutex> g(g_tm_mu);
    if (on) drop_marks_locked();
    g_tm_on = on != 0;
    return SINET_OK;
}

sinet_status timing_read(double ms[PH_COUNT], uint64_t* calls, uint64_t* stage1_launches,
                         uint64_t* window_calls) {
    std::lock_guard<std::mutex> g(g_tm_mu);
    for (int k = 0; k < PH_COUNT; ++k) ms[k] = 0.0;
    *stage1_launches = 0;
    for (const Mark& m : g_tm_marks) {
        float t = 0.f;
        sinet_status st = check_hip(hipEventSynchronize(m.b), "timing event");
        if (st == SINET_OK) st = check_hip(hipEventElapsedTime(&t, m.a, m.b), "timing event");
        if (st != SINET_OK) return st;
        ms[m.phase] += t;
        if (m.phase == PH_STAGE1) ++*stage1_launches;
    }
    *calls = g_tm_calls;
    *window_calls = g_tm_window;
    return SINET_OK;
}

// Histogram of one stream by the partitioned path (workspace given).
sinet_status run_partitioned(const PassParams& p0, uint32_t kind, const PartWs& w, int accumulate,
                             hipStream_t s) {
    PassParams p = p0;
    const bool vec = vector_ok(p, kind, true);
    PartWs wv = w;
    wv.vec = vec ? 1u : 0u;
    // directory counts (their array is padded to whole 64-bit words), far count
    // and run counter, and the dropped counters unless accumulating
    const ClearArgs c{{(unsigned long long*)w.seg_count, (unsigned long long*)w.farcount, p.dropped},
                      {((uint64_t)w.n_blocks + 1) / 2, 1, !accumulate && !w.keep_dropped && p.dropped ? 8ull : 0ull},
                      nullptr};
    sinet_status st = launch_clears(c, s);
    if (st != SINET_OK) return st;
    // runs of fewer chunks where there are too few for every CU's workgroups
    wv.run = w.n_chunks >= 8ull * device_cu_count() ? (uint32_t)kStage1Run : 1u;
    Stage1Fn f1 = pick_stage1(kind);
    const size_t lds = (kind == KK_LABEL_IN ? 0 : p.t.lds_bytes) + 8;
    if (lds + kStage1StaticLds > 160 * 1024)
        return fail(SINET_ERR_UNSUPPORTED, "table needs more LDS than a CU has");
    uint64_t grid = (uint64_t)device_cu_count() * blocks_per_cu((const void*)f1, kStage1Block, lds);
    if (grid > w.n_chunks) grid = w.n_chunks;
    if (grid < 1) grid = 1;
    {
        PhaseScope ph(PH_STAGE1, s);
        hipLaunchKernelGGL(f1, dim3((unsigned)grid), dim3(kStage1Block), lds, s, p, wv);
        st = check_hip(hipGetLastError(), "stage-1 launch");
    }
    if (st != SINET_OK) return st;
    const uint32_t nb = w.n_blocks;
    {
        PhaseScope ph(PH_INDEX, s);
        st = launch_scan_fill(wv, s);
    }
    if (st != SINET_OK) return st;
    {
        PhaseScope ph(PH_STAGE2, s);
        const uint32_t g2 = stage2_grid(nb);
        hipLaunchKernelGGL(k_stage2, dim3(g2), dim3(kStage2Block), 0, s, wv, p.count, p.hbytes,
                           p.n_bins, accumulate);
        st = check_hip(hipGetLastError(), "stage-2 launch");
    }
    if (st != SINET_OK) return st;
    // far sessions: labels are already stored, do not store them twice
    FarList far{w.farlist, w.farcount, w.farbits};
    PassParams q = p;
    q.label_out = nullptr;
    q.src_inst = nullptr;
    q.dst_inst = nullptr;
    q.dropped = nullptr;
    PhaseScope ph(PH_FAR, s);
    return launch_k_pass(q, kind, H_ATOMIC, false, far, s);
}

// ---- batch launches -----------------------------------------------------------
using BatchFn = void (*)(BatchArgs, PartWs);

static BatchFn pick_batch_stage1(uint32_t kind) {
    switch (kind) {
        case KK_SCAN: return k_batch_stage1<KK_SCAN>;
        case KK_BSEARCH: return k_batch_stage1<KK_BSEARCH>;
        case KK_TRIE: return k_batch_stage1<KK_TRIE>;
        case KK_PLA: return k_batch_stage1<KK_PLA>;
        case KK_MLP: return k_batch_stage1<KK_MLP>;
        case KK_INOUT: return k_batch_stage1_o4<KK_INOUT>;
        case KK_UNION: return k_batch_stage1_o4<KK_UNION>;
        case KK_LABEL_IN: return k_batch_stage1_o4<KK_LABEL_IN>;
        default: return nullptr;
    }
}

static BatchFn pick_batch_far(uint32_t kind) {
    switch (kind) {
        case KK_SCAN: return k_batch_far<KK_SCAN>;
        case KK_BSEARCH: return k_batch_far<KK_BSEARCH>;
        case KK_TRIE: return k_batch_far<KK_TRIE>;
        case KK_PLA: return k_batch_far<KK_PLA>;
        case KK_MLP: return k_batch_far<KK_MLP>;
        case KK_INOUT: return k_batch_far<KK_INOUT>;
        case KK_UNION: return k_batch_far<KK_UNION>;
        case KK_LABEL_IN: return k_batch_far<KK_LABEL_IN>;
        default: return nullptr;
    }
}

using LookupFn = void (*)(BatchArgs);

static LookupFn pick_batch_lookup(uint32_t kind) {
    switch (kind) {
        case KK_BSEARCH: return k_batch_lookup<KK_BSEARCH>;
        case KK_TRIE: return k_batch_lookup<KK_TRIE>;
        case KK_PLA: return k_batch_lookup<KK_PLA>;
        case KK_MLP: return k_batch_lookup<KK_MLP>;
        default: return nullptr;
    }
}

sinet_status launch_batch_lookup(uint32_t kind, const BatchArgs& a, size_t lds, uint32_t grid,
                                 hipStream_t s) {
    LookupFn fn = pick_batch_lookup(kind);
    if (!fn) return fail(SINET_ERR_UNSUPPORTED, "no batch lookup kernel for this kind");
    if (lds + sizeof(BatchStreamDev) + 16 > 160 * 1024)
        return fail(SINET_ERR_UNSUPPORTED, "batch needs more LDS than a CU has");
    const int block = lds > 40 * 1024 ? kMaxBlock : 256;
    // the window PLA's search queues (for a whole block of the largest size)
    // when they fit beside the group's largest table
    BatchArgs b = a;
    b.queue_words = 0;
    const size_t qbytes = (size_t)(kMaxBlock / 64) * kPlaQueue * 4;
    if (kind == KK_PLA && lds + qbytes + sizeof(BatchStreamDev) + 16 <= 160 * 1024) {
        b.queue_words = kPlaQueue;
        lds += qbytes;
    }
    if (grid == 0) grid = device_cu_count() * blocks_per_cu((const void*)fn, block, lds);
    hipLaunchKernelGGL(fn, dim3(grid), dim3(block), lds, s, b);
    return check_hip(hipGetLastError(), "batch lookup launch");
}

// Two workgroups per CU where the table leaves 8 KB or more for the window
// then, else one; at most 32 KB.  two: what two leave, however little.
uint32_t batch_window_words(size_t table, bool two) {
    const size_t used = kStage1StaticLds + sizeof(BatchStreamDev) + 256 + table;
    for (const size_t lds : {(size_t)80 * 1024, (size_t)160 * 1024}) {
        if (lds >= used + (two ? 0 : 8 * 1024)) return (uint32_t)((lds - used < 32 * 1024 ? lds - used : 32 * 1024) / 8);
        if (two) break;
    }
    return 0;
}

uint32_t batch_stage1_blocks_per_cu(uint32_t kind, size_t lds) {
    BatchFn fn = pick_batch_stage1(kind);
    return fn ? (uint32_t)blocks_per_cu((const void*)fn, kStage1Block, lds) : 1u;
}

sinet_status launch_batch_stage1(uint32_t kind, const BatchArgs& a, const PartWs& w, size_t lds,
                                 uint32_t grid, hipStream_t s) {
    BatchFn fn = pick_batch_stage1(kind);
    if (!fn) return fail(SINET_ERR_UNSUPPORTED, "no batch kernel for this lookup kind");
    if (lds + kStage1StaticLds + sizeof(BatchStreamDev) + 16 > 160 * 1024)
        return fail(SINET_ERR_UNSUPPORTED, "batch needs more LDS than a CU has");
    if (grid == 0) grid = device_cu_count() * blocks_per_cu((const void*)fn, kStage1Block, lds);
    hipLaunchKernelGGL(fn, dim3(grid), dim3(kStage1Block), lds, s, a, w);
    return check_hip(hipGetLastError(), "batch stage-1 launch");
}

sinet_status launch_batch_stage2(const BatchArgs& a, const PartWs& w, uint32_t n_blocks,
                                 hipStream_t s) {
    if (n_blocks == 0) return SINET_OK;
    hipLaunchKernelGGL(k_batch_stage2, dim3(stage2_grid(n_blocks)), dim3(kStage2Block), 0, s, a, w);
    return check_hip(hipGetLastError(), "batch stage-2 launch");
}

sinet_status launch_batch_order(const BatchArgs& a, const PartWs& w, hipStream_t s) {
    hipLaunchKernelGGL(k_batch_order, dim3((a.n_items + 7) / 8), dim3(256), 0, s, a, const_cast<uint4*>(a.items), w);
    return check_hip(hipGetLastError(), "batch order launch");
}

sinet_status launch_batch_aside(const BatchArgs& a, const PartWs& w, const uint2* blocks, uint32_t n_blocks,
                                hipStream_t s) {
    if (n_blocks == 0) return SINET_OK;
    const uint32_t slices = std::max(1u, 2 * device_cu_count() / n_blocks);
    hipLaunchKernelGGL(k_batch_aside, dim3(n_blocks * slices), dim3(kStage2Block), 0, s, a, w, blocks, slices);
    return check_hip(hipGetLastError(), "batch items out of order launch");
}

sinet_status launch_batch_far(uint32_t kind, const BatchArgs& a, const PartWs& w, size_t lds,
                              hipStream_t s) {
    BatchFn fn = pick_batch_far(kind);
    if (!fn) return fail(SINET_ERR_UNSUPPORTED, "no batch kernel for this lookup kind");
    const int block = lds > 40 * 1024 ? 1024 : 256;
    const uint32_t grid = device_cu_count() * blocks_per_cu((const void*)fn, block, lds);
    hipLaunchKernelGGL(fn, dim3(grid), dim3(block), lds, s, a, w);
    return check_hip(hipGetLastError(), "batch far launch");
}

sinet_status launch_zero_jobs(const ZeroJob* jobs, uint32_t n_jobs, hipStream_t s) {
    if (n_jobs == 0) return SINET_OK;
    uint32_t grid = n_jobs < 4096 ? n_jobs : 4096;
    hipLaunchKernelGGL(k_zero_jobs, dim3(grid), dim3(256), 0, s, jobs, n_jobs);
    return check_hip(hipGetLastError(), "zero launch");
}

// ---- per-device pool for the stream-ordered workspace ------------------------
static hipMemPool_t device_pool(int dev) {
    static std::mutex mu;
    static std::map<int, hipMemPool_t> pools;
    std::lock_guard<std::mutex> g(mu);
    auto it = pools.find(dev);
    if (it != pools.end()) return it->second;
    hipMemPoolProps props;
    memset(&props, 0, sizeof(props));
    props.allocType = hipMemAllocationTypePinned;
    props.location.type = hipMemLocationTypeDevice;
    props.location.id = dev;
    hipMemPool_t pool = nullptr;
    if (hipMemPoolCreate(&pool, &props) != hipSuccess) pool = nullptr;
    if (pool) {
        uint64_t thr = ~0ull;  // keep freed blocks for reuse
        (void)hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &thr);
    }
    pools[dev] = pool;
    return pool;
}

sinet_status ws_alloc(void** ptr, size_t bytes, hipStream_t s) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return check_hip(e, "hipGetDevice");
    hipMemPool_t pool = device_pool(dev);
    e = pool ? hipMallocFromPoolAsync(ptr, bytes, pool, s) : hipMallocAsync(ptr, bytes, s);
    return check_hip(e, "workspace allocation");
}

sinet_status ws_free(void* ptr, hipStream_t s) {
    return check_hip(hipFreeAsync(ptr, s), "workspace free");
}

// Which reduce the histogram calls use (sinet_set_reduce).
static std::atomic<int> g_reduce{SINET_REDUCE_AUTO};

sinet_status set_reduce(int mode) {
    if (mode != SINET_REDUCE_AUTO && mode != SINET_REDUCE_RECORDS && mode != SINET_REDUCE_WINDOW)
        return fail(SINET_ERR_INVALID_ARG, "unknown reduce");
    g_reduce.store(mode);
    return SINET_OK;
}

static Strategy hist_strategy(const PassParams& p) {
    const int mode = g_reduce.load();
    if (mode == SINET_REDUCE_AUTO || p.n_bins <= kLocalAlways) return auto_strategy(p.n, p.n_bins, p.width);
    return {mode == SINET_REDUCE_WINDOW ? R_WINDOW : R_RECORDS, false};
}

// Lookups that walk global memory (trie, learned windows, binary searches
// with a global leaf) run as their own pass before stage 1.
bool lookup_splits(const DevTable& t) {
    return t.kind == KK_TRIE || t.kind == KK_PLA || t.kind == KK_MLP ||
           (t.kind == KK_BSEARCH && t.top_log2 > 0);
}

// The columns advanced by off sessions.
static PassParams advance(const PassParams& p, uint64_t off) {
    PassParams q = p;
    q.n = p.n - off;
    auto a32 = [&](const uint32_t* x) { return x ? x + off : x; };
    q.ts = a32(p.ts);
    q.src = a32(p.src);
    q.dst = a32(p.dst);
    q.bytes = p.bytes ? p.bytes + off : nullptr;
    q.label_in = p.label_in ? p.label_in + off : nullptr;
    q.label_out = p.label_out ? p.label_out + off : nullptr;
    q.src_inst = p.src_inst ? p.src_inst + off : nullptr;
    q.dst_inst = p.dst_inst ? p.dst_inst + off : nullptr;
    return q;
}

// Sliding-window reduce (window.hip): the labels first (a lookup pass that
// stores them, unless they are given), then the window pass, the fix-up of
// the bins at the pieces' boundaries and the far path.
// With the workspace given: ws holds win_ws_bytes(n, P) bytes, then (when a
// lookup pass runs and the caller stores no labels) n bytes of labels.
static sinet_status run_window_in(const PassParams& p, uint32_t kind, int accumulate, hipStream_t s,
                                  void* ws, uint32_t P, bool timed, const uint32_t* gate = nullptr) {
    const size_t wsb = win_ws_bytes(p.n, P);
    const bool lookup = kind != KK_LABEL_IN;
    sinet_status st = SINET_OK;
    PassParams q = p;
    if (lookup) {
        PassParams lq = p;
        if (!lq.label_out) lq.label_out = (uint8_t*)ws + wsb;
        lq.pos_out = nullptr;
        FarList none{};
        PhaseScope ph(PH_LOOKUP, s, timed);
        st = launch_k_pass(lq, kind, H_NONE, vector_ok(lq, kind, false), none, s);
        q.label_in = lq.label_out;
    }
    q.label_out = nullptr;
    q.src_inst = nullptr;
    q.dst_inst = nullptr;
    WinArgs a = win_carve(ws, q, P, accumulate);
    a.gate = gate;
    if (st == SINET_OK) {
        PhaseScope ph(PH_INDEX, s, timed);
        st = win_launch_bounds(a, s);
    }
    if (st == SINET_OK) {
        PhaseScope ph(PH_STAGE1, s, timed);
        st = win_launch_main(a, s);
    }
    if (st == SINET_OK) {
        PhaseScope ph(PH_STAGE2, s, timed);
        st = win_launch_fixup(a, s);
    }
    if (st == SINET_OK) {
        PhaseScope ph(PH_FAR, s, timed);
        st = win_launch_far(a, s);
    }
    return st;
}

static size_t window_ws_total(const PassParams& p, uint32_t kind, uint32_t P) {
    const bool lookup = kind != KK_LABEL_IN;
    return win_ws_bytes(p.n, P) + (lookup && !p.label_out ? al256(p.n) : 0);
}

static sinet_status run_window(const PassParams& p, uint32_t kind, int accumulate, hipStream_t s) {
    const uint32_t P = win_pieces(p.n);
    void* ws = nullptr;
    sinet_status st = ws_alloc(&ws, window_ws_total(p, kind, P), s);
    if (st != SINET_OK) return st;
    count_window_call();
    st = run_window_in(p, kind, accumulate, s, ws, P, true);
    const sinet_status st2 = ws_free(ws, s);
    return st != SINET_OK ? st : st2;
}

using LocalFn = void (*)(PassParams, LocalArgs);

template <uint32_t KIND>
static LocalFn local_fn(bool vec, bool defer) {
    if (defer) return vec ? k_local<KIND, true, true> : k_local<KIND, false, true>;
    return vec ? k_local<KIND, true, false> : k_local<KIND, false, false>;
}

static LocalFn pick_local(uint32_t kind, bool vec, bool defer) {
    switch (kind) {
        case KK_UNION: return local_fn<KK_UNION>(vec, defer);
        case KK_INOUT: return local_fn<KK_INOUT>(vec, defer);
        case KK_LABEL_IN: return local_fn<KK_LABEL_IN>(vec, defer);
        default: return nullptr;
    }
}

template <uint32_t KIND>
static void (*aside_fn(bool vec))(PassParams, uint32_t*) {
    return vec ? k_aside<KIND, true> : k_aside<KIND, false>;
}

static sinet_status launch_aside(const PassParams& p, uint32_t kind, uint32_t* aside, hipStream_t s) {
    const bool vec = vector_ok(p, kind, true);
    const auto fn = kind == KK_UNION ? aside_fn<KK_UNION>(vec)
                                     : kind == KK_INOUT ? aside_fn<KK_INOUT>(vec) : aside_fn<KK_LABEL_IN>(vec);
    const size_t lds = kind == KK_LABEL_IN ? 0 : p.t.lds_bytes;
    const uint32_t grid = device_cu_count() * blocks_per_cu((const void*)fn, kMaxBlock, lds);
    hipLaunchKernelGGL(fn, dim3(grid), dim3(kMaxBlock), lds, s, p, aside);
    const uint32_t blocks = defer_at(aside, p.n, p.n_bins).blocks;
    const uint32_t slices = std::max(1u, 2 * device_cu_count() / blocks);
    hipLaunchKernelGGL(k_deferred, dim3(blocks * slices), dim3(kStage2Block), 0, s, p, aside, slices);
    return check_hip(hipGetLastError(), "runs out of order launch");
}

// LDS of a workgroup of the local reduce, window and table: one workgroup of
// 1,024 lanes per CU with a table, two without.
constexpr size_t kLocalLds = 156 * 1024;
constexpr size_t kLocalLdsLabels = 79 * 1024;

// Bins that its window can hold.
static uint32_t local_room(uint32_t kind, const DevTable& t) {
    const size_t tab = (kind == KK_LABEL_IN ? 0 : t.lds_bytes) + 16;
    const size_t lds = kind == KK_LABEL_IN ? kLocalLdsLabels : kLocalLds;
    return lds > tab ? (uint32_t)((lds - tab) / 32) : 0u;
}

// Label lookups that the local reduce runs itself, which leave its window room for
// the bins that always take it, whatever the order of the sessions; the others
// store their labels in a pass of their own first.
static bool local_fuses(uint32_t kind, const DevTable& t) {
    return kind == KK_LABEL_IN || ((kind == KK_UNION || kind == KK_INOUT) && local_room(kind, t) >= kLocalAlways);
}
static_assert((kLocalLdsLabels - 16) / 32 >= kLocalAlways, "labels given leave that room too");

static LocalShape shape_of(const PassParams& p, uint32_t kind) {
    return local_shape(p.n, p.n_bins, p.width, local_room(kind, p.t), device_cu_count());
}

// aside: where runs out of order go (NULL: nowhere).
static sinet_status launch_local(const PassParams& p, uint32_t kind, const LocalShape& sh,
                                 const uint32_t* gate, uint32_t* aside, hipStream_t s) {
    LocalFn fn = pick_local(kind, vector_ok(p, kind, true), aside != nullptr);
    if (!fn) return fail(SINET_ERR_UNSUPPORTED, "no kernel for this lookup kind");
    const size_t tab = (kind == KK_LABEL_IN ? 0 : p.t.lds_bytes) + 16;
    const LocalArgs a{sh.bins, sh.reps, sh.run, sh.whole ? 1u : 0u, gate, aside};
    const size_t lds = tab + (32ull * a.bins << a.reps);
    const uint64_t steps = (p.n + 4 * sh.block - 1) / (4 * sh.block);
    uint64_t grid = (uint64_t)device_cu_count() * blocks_per_cu((const void*)fn, (int)sh.block, lds);
    if (grid > steps) grid = steps;
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(sh.block), lds, s, p, a);
    return check_hip(hipGetLastError(), "local reduce launch");
}

// Bytes of the runs out of order.
static size_t defer_bytes(uint64_t n, uint32_t n_bins) {
    const DeferWs d = defer_at(nullptr, n, n_bins);
    return (size_t)(d.rec - d.any) * 4 + 4ull * d.steps * kDeferSlots;
}

// The local reduce: the output cleared, the labels stored first when the
// lookup does not run inside it (into label_out, or n bytes at `labels`), the
// runs out of order set aside when there is room for them at `aside`.
static sinet_status run_local_in(const PassParams& p, uint32_t kind, int accumulate, hipStream_t s,
                                 uint8_t* labels, uint32_t* aside, bool timed) {
    const uint64_t cells = accumulate ? 0 : 4ull * p.n_bins;
    sinet_status st = launch_clears({{p.count, p.hbytes, p.dropped, (unsigned long long*)aside},
                                     {cells, cells, !accumulate && p.dropped ? 8ull : 0ull, aside ? 1ull : 0ull}, nullptr}, s);
    PassParams q = p;
    if (st == SINET_OK && !local_fuses(kind, p.t)) {
        PassParams lq = p;
        if (!lq.label_out) lq.label_out = labels;
        FarList none{};
        PhaseScope ph(PH_LOOKUP, s, timed);
        st = launch_k_pass(lq, kind, H_NONE, vector_ok(lq, kind, false), none, s);
        q.label_in = lq.label_out;
        q.label_out = nullptr;
        kind = KK_LABEL_IN;
    }
    if (st != SINET_OK) return st;
    {
        PhaseScope ph(PH_STAGE1, s, timed);
        st = launch_local(q, kind, shape_of(q, kind), nullptr, aside, s);
    }
    if (st != SINET_OK || !aside) return st;
    PhaseScope ph(PH_STAGE2, s, timed);
    return launch_aside(q, kind, aside, s);
}

// Sessions whose labels wait in the workspace at a time, so that calls on a nearly
// full device need little of it.
constexpr uint64_t kLocalLabels = 1ull << 28;

static sinet_status run_local(const PassParams& p, uint32_t kind, int accumulate, hipStream_t s) {
    const bool fused = local_fuses(kind, p.t);
    const size_t lab = !fused && !p.label_out ? al256(std::min(p.n, kLocalLabels)) : 0;
    size_t aside = !shape_of(p, fused ? kind : (uint32_t)KK_LABEL_IN).whole && local_defers(p.n, p.n_bins)
                       ? defer_bytes(p.n, p.n_bins) : 0;
    if (aside) {  // a captured call must not come to need an allocation for it
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) {
            (void)hipGetLastError();
            aside = 0;
        }
    }
    void* ws = nullptr;
    if (aside && ws_alloc(&ws, lab + aside, s) != SINET_OK) {  // no room: only slower out of order
        (void)hipGetLastError();
        ws = nullptr;
        aside = 0;
    }
    if (lab && !ws) {
        const sinet_status st = ws_alloc(&ws, lab, s);
        if (st != SINET_OK) return st;
    }
    static_assert(kLocalLabels >= kWindowMinSessions, "calls that set runs aside are one piece");
    sinet_status st = SINET_OK;
    for (uint64_t lo = 0; st == SINET_OK && lo < p.n; lo += lab ? kLocalLabels : p.n) {
        PassParams q = advance(p, lo);
        if (lab) q.n = std::min(q.n, kLocalLabels);
        st = run_local_in(q, kind, accumulate || lo, s, (uint8_t*)ws, aside ? (uint32_t*)((char*)ws + lab) : nullptr, true);
    }
    const sinet_status st2 = ws ? ws_free(ws, s) : SINET_OK;
    return st != SINET_OK ? st : st2;
}

// The histogram of run_hist with its workspace taken from `scratch` (bytes
// long) instead of allocated: the local reduce for coarse bins (at most
// the labels), else the sliding-window reduce with as many pieces as fit.
// Records no timing events.
sinet_status run_hist_in(const PassParams& p, uint32_t mode, int accumulate, hipStream_t s,
                         void* scratch, size_t bytes) {
    const uint32_t kind = (mode & PASS_LABEL_IN) ? (uint32_t)KK_LABEL_IN : p.t.kind;
    if (p.n == 0) return SINET_OK;
    const Strategy strat = hist_strategy(p);
    if (strat.reduce == R_LOCAL)  // 2^25 sessions at most: their labels fit
        return run_local_in(p, kind, accumulate, s, (uint8_t*)scratch, nullptr, false);
    if (!accumulate) {
        const sinet_status st = launch_clear(p, 0, s);
        if (st != SINET_OK) return st;
    }
    uint32_t P = win_pieces(p.n);
    while (P > 1 && window_ws_total(p, kind, P) > bytes) P = P * 3 / 4;
    if (window_ws_total(p, kind, P) > bytes)
        return fail(SINET_ERR_INVALID_ARG, "input too large for the static scratch");
    return run_window_in(p, kind, accumulate, s, scratch, P, false);
}

// Bins that may be wide enough for the local reduce: both it and the other
// reduce are launched, behind a word that a probe sets from how far
// neighbouring sessions spread; the kernels of the one not chosen return at
// once.  The labels are stored first unless both reduces look them up alike
// (the records with a table the local reduce fuses).
static sinet_status run_probed(const PassParams& p, uint32_t kind, int accumulate, Reduce other,
                               hipStream_t s) {
    const bool fused = other == R_RECORDS && local_fuses(kind, p.t);
    const bool lookup = !fused && kind != KK_LABEL_IN;
    const uint32_t P = win_pieces(p.n);
    const size_t wsb = al256(other == R_WINDOW ? win_ws_bytes(p.n, P) : part_ws_bytes(p.n, p.n_bins));
    void* ws = nullptr;
    sinet_status st = ws_alloc(&ws, wsb + 256 + (lookup && !p.label_out ? p.n : 0), s);
    if (st != SINET_OK) return st;
    uint32_t* gate = (uint32_t*)((char*)ws + wsb);
    const uint32_t k2 = fused ? kind : (uint32_t)KK_LABEL_IN;
    const LocalShape sh = shape_of(p, k2);
    hipLaunchKernelGGL(k_local_probe, dim3(1), dim3(kMaxBlock), 0, s, p, sh.bins / 16 * 9, gate);
    st = check_hip(hipGetLastError(), "order probe launch");
    if (st == SINET_OK && !accumulate) st = launch_clear(p, 4ull * p.n_bins, s, gate);
    PassParams q = p;
    if (st == SINET_OK && lookup) {
        if (!q.label_out) q.label_out = (uint8_t*)ws + wsb + 256;
        FarList none{};
        PhaseScope ph(PH_LOOKUP, s);
        st = launch_k_pass(q, kind, H_NONE, vector_ok(q, kind, false), none, s);
        q.label_in = q.label_out;
        q.label_out = nullptr;
    }
    if (st == SINET_OK) {
        PhaseScope ph(PH_STAGE1, s);
        st = launch_local(q, k2, sh, gate, nullptr, s);
    }
    if (st == SINET_OK && other == R_WINDOW) {
        st = run_window_in(q, KK_LABEL_IN, accumulate, s, ws, P, true, gate);
    } else if (st == SINET_OK) {
        PartWs w = part_ws_carve(ws, p.n, p.n_bins);
        w.gate = gate;
        w.keep_dropped = 1;  // cleared above, and the local reduce may have added to it
        st = run_partitioned(q, k2, w, accumulate, s);
    }
    const sinet_status st2 = ws_free(ws, s);
    return st != SINET_OK ? st : st2;
}

sinet_status run_hist(const PassParams& p, uint32_t mode, int accumulate, hipStream_t s) {
    const uint32_t kind = (mode & PASS_LABEL_IN) ? (uint32_t)KK_LABEL_IN : p.t.kind;
    if (p.n == 0) return SINET_OK;
    if (!vector_ok(p, kind, true)) {
        // columns that all sit h sessions short of 16-byte alignment (slices of
        // aligned arrays): the aligned rest takes the vector path, then the first
        // h sessions are added by the atomic pass
        for (uint64_t h = 1; h < 4 && h < p.n; ++h) {
            if (!vector_ok(advance(p, h), kind, true)) continue;
            sinet_status st = run_hist(advance(p, h), mode, accumulate, s);
            if (st != SINET_OK) return st;
            PassParams head = p;
            head.n = h;
            FarList none{};
            return launch_k_pass(head, kind, H_ATOMIC, false, none, s);
        }
    }
    count_timed_call();
    const Strategy strat = hist_strategy(p);
    if (strat.reduce == R_LOCAL) return run_local(p, kind, accumulate, s);
    if (strat.probe) return run_probed(p, kind, accumulate, strat.reduce, s);
    if (strat.reduce == R_WINDOW) {
        const sinet_status st = accumulate ? SINET_OK : launch_clear(p, 0, s);
        return st == SINET_OK ? run_window(p, kind, accumulate, s) : st;
    }
    // partitioned: pieces of at most kMaxPiece sessions (32-bit slot indices)
    int acc = accumulate;
    for (uint64_t lo = 0; lo < p.n; lo += kMaxPiece) {
        PassParams q = p;
        const uint64_t len = p.n - lo < kMaxPiece ? p.n - lo : kMaxPiece;
        q.n = len;
        auto adv32 = [&](const uint32_t* a) { return a ? a + lo : a; };
        q.ts = adv32(p.ts);
        q.src = adv32(p.src);
        q.dst = adv32(p.dst);
        q.bytes = p.bytes ? p.bytes + lo : nullptr;
        q.label_in = p.label_in ? p.label_in + lo : nullptr;
        q.label_out = p.label_out ? p.label_out + lo : nullptr;
        q.src_inst = p.src_inst ? p.src_inst + lo : nullptr;
        q.dst_inst = p.dst_inst ? p.dst_inst + lo : nullptr;
        // Lookups that walk global memory (trie, learned windows, large binary
        // searches) run as their own barrier-free pass; stage 1 then reads the
        // labels (1 byte per session) instead of stalling its barriers on them.
        const bool split = kind != KK_LABEL_IN && lookup_splits(p.t);
        const size_t wsb = part_ws_bytes(len, p.n_bins);
        const size_t lab_bytes = split && !q.label_out ? ((len + 255) & ~(uint64_t)255) : 0;
        void* ws = nullptr;
        sinet_status st = ws_alloc(&ws, wsb + lab_bytes, s);
        if (st != SINET_OK) return st;
        const PartWs w = part_ws_carve(ws, len, p.n_bins);
        uint32_t k2 = kind;
        if (split) {
            PassParams lq = q;
            if (!lq.label_out) lq.label_out = (uint8_t*)ws + wsb;
            lq.pos_out = nullptr;
            FarList none{};
            PhaseScope ph(PH_LOOKUP, s);
            st = launch_k_pass(lq, kind, H_NONE, vector_ok(lq, kind, false), none, s);
            q.label_in = lq.label_out;
            q.label_out = nullptr;
            q.src_inst = nullptr;
            q.dst_inst = nullptr;
            k2 = KK_LABEL_IN;
        }
        if (st == SINET_OK) st = run_partitioned(q, k2, w, acc, s);
        sinet_status st2 = ws_free(ws, s);
        if (st != SINET_OK) return st;
        if (st2 != SINET_OK) return st2;
        acc = 1;
    }
    return SINET_OK;
}


// ---- watch-list histograms ----------------------------------------------------
using WatchFn = void (*)(WatchParams);

template <uint32_t KIND>
static WatchFn watch_fn(bool priv) {
    return priv ? k_watch<KIND, true> : k_watch<KIND, false>;
}

static WatchFn pick_watch(uint32_t kind, bool priv) {
    switch (kind) {
        case KK_SCAN: return watch_fn<KK_SCAN>(priv);
        case KK_BSEARCH: return watch_fn<KK_BSEARCH>(priv);
        case KK_TRIE: return watch_fn<KK_TRIE>(priv);
        case KK_PLA: return watch_fn<KK_PLA>(priv);
        case KK_MLP: return watch_fn<KK_MLP>(priv);
        default: return nullptr;
    }
}

sinet_status run_watch(const PassParams& p, uint32_t n_keys, int accumulate, hipStream_t s) {
    const uint64_t cells = 2ull * n_keys * p.n_bins;
    sinet_status st = SINET_OK;
    if (!accumulate) {
        st = launch_clears({{p.count, p.hbytes, p.dropped}, {cells, cells, p.dropped ? 4ull : 0ull}, nullptr}, s);
        if (st != SINET_OK) return st;
    }
    if (p.n == 0) return SINET_OK;
    const uint32_t kind = p.t.kind;
    // the table, each wave's search queue and the interval keys (interval
    // kinds), the private cells
    const bool lds_keys = kind != KK_SCAN && p.t.m <= kWatchLdsKeys;
    const size_t table_lds = (size_t)p.t.lds_bytes +
                             (kind == KK_SCAN ? 0 : 8 * kWatchQueue * (kWatchBlock / 64)) +
                             (lds_keys ? 4ull * p.t.m : 0) + 8;
    const bool priv = cells <= kWatchPrivCells && table_lds + 12 * cells + 8 <= 64 * 1024;
    WatchFn fn = pick_watch(kind, priv);
    if (!fn) return fail(SINET_ERR_UNSUPPORTED, "no watch kernel for this lookup kind");
    const size_t lds = table_lds + (priv ? 12 * cells + 8 : 0);
    if (lds > 160 * 1024) return fail(SINET_ERR_UNSUPPORTED, "table needs more LDS than a CU has");
    WatchParams w;
    w.p = p;
    w.n_keys = n_keys;
    w.vec = aligned16(p.src) && aligned16(p.dst) && aligned16(p.ts) && aligned16(p.bytes) ? 1u : 0u;
    w.lds_keys = lds_keys ? 1u : 0u;
    w.pad = 0;
    // Two workgroups per CU, or three for long inputs, though a small table leaves
    // room for four: each stages the table and each of its waves ends with a
    // search of what it holds.  1.3e7 sessions took 48.3 us with four, 44.6 with
    // three, 41.6 with two; 4e7 90.0, 75.2, 75.8; 4e8 744, 673, 678.
    const uint32_t most = p.n < (1ull << 26) ? 2u : 3u;
    const uint32_t per_cu = std::min(most, (uint32_t)blocks_per_cu((const void*)fn, kWatchBlock, lds));
    uint64_t grid = (uint64_t)device_cu_count() * per_cu;
    const uint64_t tiles = ((p.n + 3) / 4 + kWatchBlock - 1) / kWatchBlock;
    if (grid > tiles) grid = tiles;
    if (grid < 1) grid = 1;
    count_timed_call();
    PhaseScope ph(PH_LOOKUP, s);
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(kWatchBlock), lds, s, w);
    return check_hip(hipGetLastError(), "watch kernel launch");
}

}  // namespace sinet
