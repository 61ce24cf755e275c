// The local reduce's shape (the header the library includes) over sessions,
// bins, widths and room: the copies fit, a run's counts fit their 17 bits, a
// moving window keeps the time that its rule promises, and a run's advance
// leaves most of it to the time jitter.  Then the reduce that calls take.
#include <cstdio>
#include <initializer_list>

#include "local_shape.h"

using namespace sinet;

int main() {
    unsigned long long bad = 0, seen = 0, moving = 0;
    for (uint64_t n = 1; n < 2000000000ull; n = n * 3 + 1)
        for (uint32_t n_bins = 1; n_bins < 90000000u; n_bins = n_bins * 2 + n_bins / 3 + 1)
            for (uint32_t width : {1u, 4u, 7u, 10u, 20u, 47u, 48u, 50u, 100u, 333u, 1000u, 60000u, 86400000u})
                for (uint32_t cap : {2047u, 2527u, 2943u, 4700u}) {
                    const LocalShape s = local_shape(n, n_bins, width, cap, 256);
                    const uint64_t step = 4ull * s.block, per_bin = n / n_bins + 1;
                    bool ok = s.bins >= 1 && ((uint64_t)s.bins << s.reps) <= cap && s.run >= 1 &&
                              s.run * step <= kLocalRun;
                    if (s.whole) {
                        ok = ok && s.bins == n_bins;
                    } else {
                        ++moving;
                        const uint64_t full = (uint64_t)cap * width, span = (uint64_t)s.bins * width;
                        ok = ok && s.bins <= n_bins && (span >= kLocalSureSpan || span == full) &&
                             (s.run == 1 || (s.run * step) / per_bin <= (uint64_t)s.bins * 3 / 8);
                    }
                    ++seen;
                    if (!ok && ++bad <= 10)
                        printf("n %llu bins %u width %u cap %u: window %u reps %u run %u block %u\n",
                               (unsigned long long)n, n_bins, width, cap, s.bins, s.reps, s.run, s.block);
                }
    // calls: sessions, bins, width; the reduce, probed, runs out of order set aside
    struct { uint64_t n; uint32_t n_bins, width; Reduce r; bool probe, defers; } routes[] = {
        {5, 2048, 1, R_LOCAL, false, false},                  // the window holds every bin
        {4000000, 3000, 1, R_RECORDS, false, false},          // narrower than any jitter
        {4000000, 3000, 10, R_RECORDS, true, false},
        {400000000, 360000, 10, R_WINDOW, true, false},
        {100000000, 43200, 1000, R_LOCAL, false, true},
        {100000000, 65536, 48, R_LOCAL, false, true},
        {100000000, 86400, 1000, R_LOCAL, false, false},      // more blocks than a wave scans
        {60000000, 43200, 1000, R_LOCAL, false, false},       // too short to hide a launch
        {400000000, 43200, 1000, R_LOCAL, false, false},      // too much room
        {1600000000, 86400000, 1, R_WINDOW, false, false},
        {100000000, 86400000, 1, R_RECORDS, false, false},
    };
    for (const auto& t : routes) {
        const Strategy g = auto_strategy(t.n, t.n_bins, t.width);
        const bool defers = g.reduce == R_LOCAL && t.n_bins > kLocalAlways && local_defers(t.n, t.n_bins);
        if (g.reduce != t.r || g.probe != t.probe || defers != t.defers) {
            ++bad;
            printf("n %llu bins %u width %u: reduce %d probe %d aside %d\n", (unsigned long long)t.n, t.n_bins,
                   t.width, (int)g.reduce, (int)g.probe, (int)defers);
        }
    }
    printf("shapes %llu moving %llu bad %llu\n", seen, moving, bad);
    return bad || !moving ? 1 : 0;
}
