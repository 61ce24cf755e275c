// Institution index: the institution of the longest matching prefix of an
// address (Algorithm 1 over the whole table), from a short search in LDS and
// two reads of tables that L2 holds.
//
// The address space is cut where the institution changes (neighbouring
// intervals with the same institution are one): boundaries with the value MI
// from each on (SINET_NO_INST outside every prefix).
//   groups  one word per 16 consecutive /16 blocks: bit k says that block k has
//           a record (something other than "outside" somewhere in it), bits 16
//           to 31 hold the number of records in all earlier groups;
//   first   per record its first leaf (a record's leaves are consecutive, and
//           the next record's first leaf ends them);
//   sample  per leaf its first boundary;
//   leaves  coded, with few distinct institutions (at most 4,095, ids below
//           2^20): 32 bytes, up to seven boundaries and the 16-bit codes of
//           the eight institutions between them (0: outside), for a dictionary
//           that LDS holds; else 16 bytes: the index into MI before the leaf's
//           first boundary, then up to six boundaries.
// Boundaries lie strictly inside the block and are kept as their 16-bit
// offsets less one, ascending, padded with 0xFFFF: b <= x is b - 1 < x, which
// no pad satisfies.  Leaves hold equal numbers of boundaries rather than equal
// parts of the block because prefixes cluster: parts of at most six boundaries
// took 254,000 16-byte slots for the 200,000-prefix table (4 MB, the whole L2
// of an XCD) and still left 30 % of its boundaries to a search.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

namespace sinet {

constexpr uint32_t kInstGroups = 65536 / 16;
constexpr uint32_t kInstLeaf = 6;        // boundaries of a leaf with an index into MI
constexpr uint32_t kInstLeafCoded = 7;   // boundaries of a leaf with codes
constexpr uint32_t kInstDictMax = 4096;  // dictionary words (16 KB of LDS)
constexpr uint32_t kInstIdMax = 1u << 20;  // end of the ids that take codes
constexpr uint32_t kInstNone = 0xFFFFFFFFu;

struct InstIndex {
    std::vector<uint32_t> groups;  // [kInstGroups]
    std::vector<uint32_t> first;   // [records + 2]: the leaf count, twice, after the records
    std::vector<uint16_t> sample;  // [leaves + 1]
    std::vector<uint32_t> leaves;  // [4 or 8 words * (leaves + 1)]: a pad leaf after the last
    std::vector<uint32_t> MI;      // coded: the dictionary
    bool coded = false;
    uint32_t steps = 0;            // halvings that search the longest record's leaves
};

// From the table's intervals (B ascending from 0, owner row + 1 or 0) and the
// rows' institutions.
inline void build_inst_index(const std::vector<uint32_t>& B, const std::vector<uint32_t>& owner,
                             const uint32_t* inst, InstIndex& ix) {
    std::vector<uint32_t> MB;
    MB.reserve(B.size());
    ix.MI.reserve(B.size());
    for (size_t j = 0; j < B.size(); ++j) {
        const uint32_t v = owner[j] ? inst[owner[j] - 1] : kInstNone;
        if (ix.MI.empty() || ix.MI.back() != v) {
            MB.push_back(B[j]);
            ix.MI.push_back(v);
        }
    }
    // codes in order of first use (0: outside), for ids that a small array maps
    uint32_t max_id = 0;
    for (const uint32_t v : ix.MI)
        if (v != kInstNone && v > max_id) max_id = v;
    ix.coded = max_id < kInstIdMax;
    std::vector<uint16_t> code_of(ix.coded ? max_id + 1 : 0, 0);
    std::vector<uint32_t> dict{kInstNone};
    for (size_t j = 0; j < ix.MI.size() && ix.coded; ++j) {
        const uint32_t v = ix.MI[j];
        if (v == kInstNone) continue;
        if (code_of[v]) continue;
        ix.coded = dict.size() < kInstDictMax;
        code_of[v] = (uint16_t)dict.size();
        dict.push_back(v);
    }
    auto code = [&](uint32_t v) -> uint16_t { return v == kInstNone ? 0 : code_of[v]; };
    const size_t cap = ix.coded ? kInstLeafCoded : kInstLeaf;
    ix.groups.assign(kInstGroups, 0);
    auto leaf = [&](uint32_t j0, const uint32_t* b, size_t n) {
        uint16_t h[16] = {};  // boundaries, then codes
        for (size_t i = 0; i < 8; ++i) h[i] = i < n ? (uint16_t)((b[i] & 0xFFFFu) - 1u) : 0xFFFFu;
        ix.sample.push_back(h[0]);
        if (ix.coded)
            for (size_t i = 0; i < 8; ++i) h[8 + i] = code(ix.MI[j0 + (i < n ? i : n)]);
        uint32_t w[8];
        for (size_t i = 0; i < 8; ++i) w[i] = (uint32_t)h[2 * i] | (uint32_t)h[2 * i + 1] << 16;
        if (!ix.coded) w[3] = w[2], w[2] = w[1], w[1] = w[0], w[0] = j0;
        ix.leaves.insert(ix.leaves.end(), w, w + (ix.coded ? 8 : 4));
    };
    ix.first.reserve(65536 + 2);
    ix.sample.reserve(65536 + MB.size() / cap);
    ix.leaves.reserve(8 * (65536 + MB.size() / cap));
    uint32_t most = 1;
    size_t u = 0;  // boundaries at or below the block's first address
    for (uint32_t k = 0; k < 65536; ++k) {
        if ((k & 15u) == 0) ix.groups[k >> 4] = (uint32_t)ix.first.size() << 16;
        while (u < MB.size() && MB[u] <= k << 16) ++u;
        size_t e = u;  // boundaries [u, e) lie strictly inside the block
        while (e < MB.size() && (MB[e] >> 16) == k) ++e;
        if (u == e && ix.MI[u - 1] == kInstNone) continue;
        ix.groups[k >> 4] |= 1u << (k & 15u);
        ix.first.push_back((uint32_t)ix.sample.size());
        size_t i = u;
        do {
            const size_t n = e - i < cap ? e - i : cap;
            leaf((uint32_t)(i - 1), MB.data() + i, n);
            i += n;
        } while (i < e);
        const uint32_t n = (uint32_t)ix.sample.size() - ix.first.back();
        if (n > most) most = n;
        u = e;
    }
    ix.first.push_back((uint32_t)ix.sample.size());
    ix.first.push_back((uint32_t)ix.sample.size());
    leaf(0, nullptr, 0);  // read, never used, by addresses without a record
    for (; most > 1; most -= most >> 1) ++ix.steps;
    if (ix.coded) ix.MI = dict;
}

// The last of n leaves from lo on whose first boundary is at or below offset
// x (the first leaf when none is), in `steps` halvings.
template <class Sample>
__host__ __device__ inline uint32_t inst_leaf_of(const Sample& sample, uint32_t lo, uint32_t n,
                                                 uint32_t steps, uint32_t x) {
    for (uint32_t s = 0; s < steps; ++s) {
        const uint32_t half = n >> 1;
        lo = sample(lo + half) < x ? lo + half : lo;
        n -= half;
    }
    return lo;
}

// Per half of a and b: the smaller of 1 and what x exceeds the stored boundary
// by (0 when it does not), that is 1 when the boundary is at or below x.  The
// two packed instructions are written out because the compiler otherwise
// splits the halves into compares and selects (about twice the instructions).
__host__ __device__ inline uint32_t inst_below(uint32_t word, uint32_t xx) {
#ifdef __HIP_DEVICE_COMPILE__
    uint32_t d, r;
    asm("v_pk_sub_u16 %0, %1, %2 clamp" : "=v"(d) : "v"(xx), "v"(word));
    asm("v_pk_min_u16 %0, %1, %2" : "=v"(r) : "v"(d), "s"(0x00010001u));
    return r;
#else
    return ((word & 0xFFFFu) < (xx & 0xFFFFu) ? 1u : 0u) | ((word >> 16) < (xx >> 16) ? 0x10000u : 0u);
#endif
}

// The index into MI of offset x in a leaf (four words).
__host__ __device__ inline uint32_t inst_in_leaf(const uint32_t* w, uint32_t x) {
    const uint32_t xx = x | x << 16;
    uint32_t c = inst_below(w[1], xx);  // counts of the even and the odd places (at most 3 each)
#pragma unroll
    for (int k = 2; k < 4; ++k) c += inst_below(w[k], xx);
    return w[0] + (c & 0xFFFFu) + (c >> 16);
}

// The code of offset x in a coded leaf (eight words).
__host__ __device__ inline uint32_t inst_code_in_leaf(const uint32_t* w, uint32_t x) {
    const uint32_t xx = x | x << 16;
    uint32_t c = inst_below(w[0], xx);
#pragma unroll
    for (int k = 1; k < 4; ++k) c += inst_below(w[k], xx);
    c = (c & 0xFFFFu) + (c >> 16);  // 0..7
    const uint32_t lo = c & 2u ? w[5] : w[4], hi = c & 2u ? w[7] : w[6];
    return ((c & 4u ? hi : lo) >> (16u * (c & 1u))) & 0xFFFFu;
}

}  // namespace sinet
