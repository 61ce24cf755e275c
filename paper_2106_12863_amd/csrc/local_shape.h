// Which reduce a histogram call takes, and the shape of its local reduce
// (k_local): the window of bins that a workgroup keeps in LDS, its copies, and
// how many sessions it takes between two flushes.  One function decides the
// shape, for the launch and for the probe that asks whether the sessions' order
// allows it.
#pragma once

#include <stdint.h>

namespace sinet {

constexpr uint32_t kLocalRun = (1u << 17) - 1u;  // sessions of a run at most (17-bit counts)
constexpr uint32_t kLocalSureSpan = 120000;      // time (ms) that the copies leave a window

constexpr uint32_t kLocalAlways = 2048;          // bins that always take the local reduce

// The local reduce is a candidate from this many sessions per bin on.  Fewer
// leave it little to add up in LDS before its device atomics: 1e8 sessions of a
// day took 1.11 ms with 12 sessions per bin, 0.76 with 23, 0.60 with 58 and 0.44
// with 116, the records 0.89-0.93 ms each.  Small calls gain before that (4e6
// sessions, 11 per bin: 62 against 91 us) but would need a probe of their order.
constexpr uint64_t kLocalMinPerBin = 16;

// Width from which the window spans kLocalSureSpan whatever its copies
// (local_shape): up to about +-1 minute of disorder.  With narrower bins a probe
// looks first: with +-5 s of jitter 4e8 sessions at 4 ms per bin took 13.3 ms
// with the local reduce, whose window they leave, 1.45 ms with the sliding
// window; at 10 ms per bin 1.71 against 15.6 ms.
constexpr uint32_t kLocalSureWidth = 48;
// Width below which not even +-5 s of jitter fits the window: no probe.
constexpr uint32_t kLocalMinWidth = 4;

// The window reduce has about 0.7 ms of fixed cost per call (its pieces'
// boundary fix-up and far pass, and the write-out of bins its few sessions
// leave behind); on the day shape with 86.4 M 1-ms bins it was measured at
// 2.25 ms against 1.82 ms for the records with 1e8 sessions and 3.38 against
// 3.70 ms with 4e8, a crossover near 2.7e8 sessions.
constexpr uint64_t kWindowMinSessions = 1ull << 28;

// Calls of the local reduce with a moving window that set runs out of order
// aside (k_local's third form).  From the line at which what that costs sessions
// in order, 10 us, is a twenty-fifth of the call; up to the window reduce's,
// because the room for the records is 5 bytes a session (and from there on
// shuffled input was never faster: 4e8 sessions into 65,536 bins 33.1 ms, 36.1
// with the window reduce); and up to 64 blocks of bins.  Those are the bins that
// the records take in any order, so that the local reduce is the slower one for
// shuffled sessions: shorter calls 1.1 to 2 times (1.6e7 into 65,536 bins 1.34
// against 0.79 ms), more bins 1.2 times (86,400: 8.47 against 7.05).
constexpr uint64_t kDeferMin = 90000000;
constexpr uint32_t kDeferMaxBins = 64 * 1024;
inline bool local_defers(uint64_t n, uint32_t n_bins) {
    return n >= kDeferMin && n < kWindowMinSessions && n_bins <= kDeferMaxBins;
}

enum Reduce { R_LOCAL, R_RECORDS, R_WINDOW };

struct Strategy {
    Reduce reduce;  // R_RECORDS or R_WINDOW, or R_LOCAL when the local reduce is sure
    bool probe;     // the local reduce runs instead if the sessions' order allows it
};

// The reduce of n sessions into n_bins bins of `width` ms.
inline Strategy auto_strategy(uint64_t n, uint32_t n_bins, uint32_t width) {
    if (n_bins <= kLocalAlways) return {R_LOCAL, false};
    const Reduce other = n >= kWindowMinSessions ? R_WINDOW : R_RECORDS;
    if (n / n_bins < kLocalMinPerBin || width < kLocalMinWidth) return {other, false};
    if (width >= kLocalSureWidth) return {R_LOCAL, false};
    return {other, true};
}

struct LocalShape {
    uint32_t bins;   // bins of the window
    uint32_t reps;   // log2 of the window's copies
    uint32_t block;  // lanes of a workgroup; a step is four sessions a lane
    uint32_t run;    // steps between two flushes
    bool whole;      // the window is the whole histogram
};

// n sessions into n_bins bins of `width` ms with room for `cap` bins in LDS.
//
// The copies (sessions of one bin meet in fewer words) divide the room, so they
// stop where the window would no longer span kLocalSureSpan ms, or all of the
// room if that spans less: a log whose times are out of order by up to +-J fits
// when 2 J and a run's advance fit.  Without that line 2e8 sessions of ten
// minutes in 10-ms bins, +-5 s, took two doublings and a window of 631 of 2,527
// bins, which 42 % of them missed: 7.72 ms, 0.51 with it (records 3.17); 4e8 of
// an hour in 50-ms bins 20.2 against 0.99 ms at +-30 s, 30.3 against 1.35 ms at
// +-1 minute (records 5.99 and 6.76), and 0.93 ms either way at +-5 s.
inline LocalShape local_shape(uint64_t n, uint32_t n_bins, uint32_t width, uint32_t cap, uint32_t cus) {
    LocalShape s{};
    // small inputs: smaller steps, so that more CUs take part
    s.block = n >= 2048ull * cus ? 1024 : 256;
    const uint32_t step = 4 * s.block, most = kLocalRun / step;
    s.whole = n_bins <= cap;
    s.run = most;
    const uint64_t per_bin = n / n_bins + 1;
    uint64_t want = n_bins;  // bins the copies must each hold
    if (!s.whole) {
        // a run moves forward by at most 3/8 of the window, the rest is for the
        // time jitter; the copies hold eight times a full run's advance
        const uint64_t fit = (uint64_t)cap * 3 / 8 * per_bin / step;
        s.run = (uint32_t)(fit < 1 ? 1 : fit < most ? fit : most);
        want = 8 * ((uint64_t)kLocalRun / per_bin) + 256;
        if (want * width < kLocalSureSpan) want = (kLocalSureSpan + width - 1) / width;
    }
    // copies while they fit and hold fewer words than the workgroup has sessions
    const uint64_t steps = (n + step - 1) / step;
    const uint64_t mine = n / (steps < cus ? steps : cus);
    while (s.reps < 4 && want << (s.reps + 1) <= cap && want << (s.reps + 3) <= mine) ++s.reps;
    s.bins = s.whole ? n_bins : cap >> s.reps;
    return s;
}

}  // namespace sinet
