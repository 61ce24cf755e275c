// Host check of the institution index (paper_2106_12863_amd/csrc/inst_index.h):
// an address's record, leaf and MI entry against the owner of its interval by
// plain search, for interval sets that leave leaves nearly empty, that put many
// leaves into a /16 block, that fill a block with every address a boundary, or that cover the whole space.  Addresses: uniform, each
// boundary +-2, and every address of one dense block.  Exit status 0 when every
// lookup agrees.
#include "inst_index.h"
#include <algorithm>
#include <cstdio>
#include <random>
using namespace sinet;
int main() {
    std::mt19937_64 rng(11);
    long bad = 0, checked = 0, searched = 0, coded = 0, indexed = 0;
    for (int trial = 0; trial < 40; ++trial) {
        std::vector<uint32_t> B{0};
        const int kind = trial % 5, nb = kind == 4 ? 1 : 1000 + (int)(rng() % 8000);
        for (int i = 0; i < nb; ++i) {
            if (kind == 0) B.push_back((uint32_t)rng());                                        // sparse
            else if (kind == 1) B.push_back((uint32_t)(rng() % 30) << 16 | (uint32_t)(rng() & 0xFFFF));  // dense blocks
            else if (kind == 2) B.push_back(0x0A0B0000u | (uint32_t)(rng() % 300));              // dense part
            else if (kind == 3) B.push_back((uint32_t)(rng() % 65536) << 16 | (uint32_t)(rng() % 3) * 0x8000u);
        }
        if (trial == 9) for (uint32_t x = 0; x < 65536; ++x) B.push_back(0xFFFF0000u | x);       // all of a block
        std::sort(B.begin(), B.end());
        B.erase(std::unique(B.begin(), B.end()), B.end());
        std::vector<uint32_t> owner(B.size()), inst(trial % 2 ? 64 : 20000);  // few institutions, or more than the codes take
        for (uint32_t& v : inst) v = (uint32_t)(rng() % (inst.size() / 2 + 8)) * 50u;
        for (uint32_t& o : owner) o = (uint32_t)(rng() % (inst.size() + 1));
        if (trial == 4) owner[0] = 0;   // nothing at all
        if (trial == 9) for (size_t j = 1; j < owner.size(); ++j) if (B[j] >= 0xFFFF0000u) owner[j] = 1 + (j & 1);
        inst[0] = 77; inst[1] = 78;
        InstIndex ix;
        build_inst_index(B, owner, inst.data(), ix);
        (ix.coded ? coded : indexed)++;
        auto check = [&](uint32_t a) {
            const size_t j = std::upper_bound(B.begin(), B.end(), a) - B.begin() - 1;
            const uint32_t want = owner[j] ? inst[owner[j] - 1] : kInstNone;
            const uint32_t w = ix.groups[a >> 20], k = (a >> 16) & 15u;
            uint32_t got = kInstNone;
            if ((w >> k) & 1u) {
                const uint32_t r = (w >> 16) + __builtin_popcount(w & ((1u << k) - 1u));
                const uint32_t f = ix.first[r], n = ix.first[r + 1] - f, x = a & 0xFFFFu;
                searched += n > 1;
                const uint32_t at = inst_leaf_of([&](uint32_t i) { return (uint32_t)ix.sample[i]; }, f, n, ix.steps, x);
                got = ix.MI[ix.coded ? inst_code_in_leaf(&ix.leaves[8 * (size_t)at], x)
                                     : inst_in_leaf(&ix.leaves[4 * (size_t)at], x)];
            }
            ++checked;
            if (got != want && ++bad < 6) printf("bad trial %d a=%08x got %u want %u\n", trial, a, got, want);
        };
        for (uint32_t b : B) for (int d = -2; d <= 2; ++d) check(b + (uint32_t)d);
        for (int i = 0; i < 200000; ++i) check((uint32_t)rng());
        for (uint32_t x = 0; x < 65536; ++x) { check(0x0A0B0000u | x); check(0xFFFF0000u | x); check(0x00050000u | x); }
    }
    printf("checked %ld searched %ld bad %ld\n", checked, searched, bad);
    return bad != 0 || searched == 0 || coded == 0 || indexed == 0;
}
