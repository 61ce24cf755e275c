// Shape of a call's local reduce (k_local): the window of bins that a workgroup
// keeps in LDS, its copies, and how many sessions it takes between two flushes.
// One function decides it, for the launch and for the probe that asks whether
// the sessions' order allows it.
#pragma once

#include <stdint.h>

namespace sinet {

constexpr uint32_t kLocalRun = (1u << 17) - 1u;  // sessions of a run at most (17-bit counts)
constexpr uint32_t kLocalSureSpan = 120000;      // time (ms) that the copies leave a window

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
