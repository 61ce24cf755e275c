// Institution ids of both ends of every session through the institution
// index (inst_index.h).
//
// HBM moves 8 B/session in and up to 9 B out (0.32 ms for 1e8 sessions at the
// rate of a large copy); every address in a /16 block with a record also costs
// one random read of an L2-resident table (two without codes).  Random 4- or
// 16-byte reads of a 1-4 MB table run at 2.65e11 reads/s on the device, of a
// 16 MB one at 0.8e11, and that rate, not latency, is most of what is left (vector
// issue is busy 67 % of the time, LDS with conflicts 38 %): deferring the
// institution reads by an iteration, 24 or 32 waves per CU instead of 16, or a
// common address for the lanes without a record changed nothing (0.89-0.95 ms).
// So everything but the leaf is kept in LDS, and with few distinct institutions
// the leaf itself holds their codes.  1e8 sessions against 200,000 prefixes, both
// ids and the label: 4.08 ms by the binary search over the intervals (14 LDS
// steps, 4 dependent global reads, then the owner and its id), 0.89 ms with an
// index into MI in the leaf, 0.75 ms with codes.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "inst_index.h"
#include "pass_common.h"
#include "sinet_internal.h"

namespace sinet {
namespace {

constexpr int kInstBlock = 1024;
// LDS of one workgroup; a table whose records and samples do not fit reads
// them through L2 (their 16-bit form in LDS also holds at most 65,536 leaves).
constexpr size_t kInstLdsMax = 156 * 1024;

struct InstArgs {
    InstDev x;
    const uint32_t* src;
    const uint32_t* dst;
    uint8_t* label;
    uint32_t* src_inst;
    uint32_t* dst_inst;
    uint64_t n;
};

template <int N, bool CODED, bool LDS>
__device__ __forceinline__ void inst_lookup(const InstDev& x, const uint32_t* grp, const uint32_t* dict,
                                            const uint16_t* first, const uint16_t* sample,
                                            const uint32_t* a, uint32_t* out) {
    uint32_t g[N];
    uint32_t need = 0, lo[N], n[N];
#pragma unroll
    for (int q = 0; q < N; ++q) g[q] = grp[a[q] >> 20];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const uint32_t k = (a[q] >> 16) & 15u;
        need |= ((g[q] >> k) & 1u) << q;
        // at most the word after the last record's, which an address without
        // a record reads in vain
        const uint32_t r = (g[q] >> 16) + (uint32_t)__builtin_popcount(__builtin_amdgcn_ubfe(g[q], 0u, k));
        lo[q] = LDS ? first[r] : *glob(x.first + r);
        n[q] = (LDS ? first[r + 1] : *glob(x.first + r + 1)) - lo[q];
    }
    for (uint32_t s = 0; s < x.steps; ++s) {  // inst_leaf_of, all addresses in lockstep
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const uint32_t half = n[q] >> 1, at = lo[q] + half;
            const uint32_t v = LDS ? sample[at] : *glob(x.sample + at);
            lo[q] = v < (a[q] & 0xFFFFu) ? at : lo[q];
            n[q] -= half;
        }
    }
    // every leaf read is issued before any is used; addresses without a record
    // issue none
    const u32x4_t* leaves = reinterpret_cast<const u32x4_t*>(x.leaves);
    if constexpr (CODED) {
        u32x4_t v[N], w[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            v[q] = w[q] = u32x4_t{0u, 0u, 0u, 0u};  // code 0
            if ((need >> q) & 1u) {
                v[q] = *glob(leaves + 2u * lo[q]);
                w[q] = *glob(leaves + 2u * lo[q] + 1u);
            }
        }
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const uint32_t leaf[8] = {v[q].x, v[q].y, v[q].z, v[q].w, w[q].x, w[q].y, w[q].z, w[q].w};
            out[q] = dict[inst_code_in_leaf(leaf, a[q] & 0xFFFFu)];
        }
    } else {
        u32x4_t v[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            v[q] = u32x4_t{0u, 0u, 0u, 0u};
            if ((need >> q) & 1u) v[q] = *glob(leaves + lo[q]);
        }
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const uint32_t leaf[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
            const uint32_t j = inst_in_leaf(leaf, a[q] & 0xFFFFu);
            out[q] = kInstNone;
            if ((need >> q) & 1u) out[q] = *glob(x.MI + j);
        }
    }
}

template <bool CODED, bool LDS, bool VEC>
__global__ void __launch_bounds__(kInstBlock) k_inst(InstArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    for (uint32_t k = threadIdx.x; k < kInstGroups; k += kInstBlock) lds[k] = *glob(a.x.groups + k);
    uint32_t* dict = lds + kInstGroups;
    uint16_t* first = reinterpret_cast<uint16_t*>(dict + (CODED ? a.x.n_dict : 0u));
    uint16_t* sample = first + a.x.n_first;
    if constexpr (CODED)
        for (uint32_t k = threadIdx.x; k < a.x.n_dict; k += kInstBlock) dict[k] = *glob(a.x.MI + k);
    if constexpr (LDS) {
        for (uint32_t k = threadIdx.x; k < a.x.n_first; k += kInstBlock) first[k] = (uint16_t)*glob(a.x.first + k);
        for (uint32_t k = threadIdx.x; k < a.x.n_sample; k += kInstBlock) sample[k] = *glob(a.x.sample + k);
    }
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * kInstBlock * 4;
    uint64_t i = ((uint64_t)blockIdx.x * kInstBlock + threadIdx.x) * 4;
    auto load = [&](const uint32_t* q, uint64_t at) -> uint4 {  // streamed once: nontemporal
        const u32x4_t v = __builtin_nontemporal_load(glob(reinterpret_cast<const u32x4_t*>(q + at)));
        return make_uint4(v.x, v.y, v.z, v.w);
    };
    uint4 ns = make_uint4(0u, 0u, 0u, 0u), nd = ns;
    if (VEC && i + 4 <= a.n) {
        ns = load(a.src, i);
        nd = load(a.dst, i);
    }
    for (; i < a.n; i += stride) {
        const bool full = VEC && i + 4 <= a.n;
        uint32_t ad[8] = {ns.x, ns.y, ns.z, ns.w, nd.x, nd.y, nd.z, nd.w};
        if (!full) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                ad[k] = i + k < a.n ? *glob(a.src + i + k) : 0u;
                ad[4 + k] = i + k < a.n ? *glob(a.dst + i + k) : 0u;
            }
        }
        if (VEC && i + stride + 4 <= a.n) {
            ns = load(a.src, i + stride);
            nd = load(a.dst, i + stride);
        }
        uint32_t id[8], lab = 0;
        inst_lookup<8, CODED, LDS>(a.x, lds, dict, first, sample, ad, id);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            lab |= ((id[k] != kInstNone ? 1u : 0u) | (id[4 + k] != kInstNone ? 2u : 0u)) << (8 * k);
        if (full) {
            if (a.label) __builtin_nontemporal_store(lab, glob(reinterpret_cast<uint32_t*>(a.label + i)));
            if (a.src_inst)
                __builtin_nontemporal_store(u32x4_t{id[0], id[1], id[2], id[3]},
                                            glob(reinterpret_cast<u32x4_t*>(a.src_inst + i)));
            if (a.dst_inst)
                __builtin_nontemporal_store(u32x4_t{id[4], id[5], id[6], id[7]},
                                            glob(reinterpret_cast<u32x4_t*>(a.dst_inst + i)));
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (i + k >= a.n) continue;
                if (a.label) *glob(a.label + i + k) = (uint8_t)(lab >> (8 * k));
                if (a.src_inst) *glob(a.src_inst + i + k) = id[k];
                if (a.dst_inst) *glob(a.dst_inst + i + k) = id[4 + k];
            }
        }
    }
}

// LDS of a workgroup with the records and samples in it, or 0 when they do not fit.
size_t inst_lds(const InstDev& x) {
    const size_t lds = 4ull * (kInstGroups + x.n_dict) + 2ull * (x.n_first + x.n_sample);
    return lds <= kInstLdsMax && x.n_sample <= 65536 ? lds : 0;
}

}  // namespace

// Where the records and samples fit LDS the index is the faster one for every
// kind.  Where each step of the search reads L2 instead, it depends (5e7 sessions,
// both ids and the label):
//   a trie (at most three reads) and a PLA whose windows are 16 boundaries are
//   faster themselves: 400,000 clustered prefixes 3.12 ms by the index, 1.65 by the
//   trie, 1e6 3.80 and 2.67; 100,000 random /24 1.80, 1.76 and 1.25 by the PLA;
//   the other searches lose where the index takes few steps (70,000 random /24, two:
//   1.70 against 2.01 ms; 1e6, four: 2.96 against 8.41) or the table is large
//   (600,000 clustered prefixes, 726,000 boundaries, eight steps: 3.45 against 3.97;
//   1e6 3.83 against 4.99), else they win (400,000, 485,000 boundaries, eight: 3.12
//   against 2.72).
bool inst_pays(const InstDev& x, uint32_t kind, bool window, uint32_t m) {
    if (!x.groups) return false;
    if (inst_lds(x)) return true;
    if (kind == SINET_LOOKUP_TRIE || (kind == SINET_LOOKUP_LEARNED_PLA && window)) return false;
    return x.steps <= 4 || m >= (1u << 19);
}

sinet_status run_inst(const InstDev& x, const uint32_t* src, const uint32_t* dst, uint64_t n,
                      uint8_t* label, uint32_t* src_inst, uint32_t* dst_inst, hipStream_t s) {
    const InstArgs a{x, src, dst, label, src_inst, dst_inst, n};
    const bool vec = (((uintptr_t)src | (uintptr_t)dst | (uintptr_t)src_inst | (uintptr_t)dst_inst) & 15u) == 0 &&
                     ((uintptr_t)label & 3u) == 0;
    const bool in_lds = inst_lds(x) != 0;
    const size_t lds = in_lds ? inst_lds(x) : 4ull * (kInstGroups + x.n_dict);
    auto pick = [&](auto coded) {
        constexpr bool C = decltype(coded)::value;
        return in_lds ? (vec ? k_inst<C, true, true> : k_inst<C, true, false>)
                      : (vec ? k_inst<C, false, true> : k_inst<C, false, false>);
    };
    auto fn = x.n_dict ? pick(std::true_type{}) : pick(std::false_type{});
    uint64_t grid = (uint64_t)device_cu_count() * blocks_per_cu((const void*)fn, kInstBlock, lds);
    const uint64_t tiles = (n + 4 * kInstBlock - 1) / (4 * kInstBlock);
    if (grid > tiles) grid = tiles;
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(kInstBlock), lds, s, a);
    return check_hip(hipGetLastError(), "institution kernel launch");
}

}  // namespace sinet
