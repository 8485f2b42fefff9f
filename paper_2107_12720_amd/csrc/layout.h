// layout.h -- how many entries the per-vertex working arrays hold and how
// they are shared out: plain arithmetic, no HIP, so that it is checked on the
// host for every size a kept context may meet.
#pragma once
#include <cstdint>

namespace trim {

// Vertices a context's arrays are sized for when a call of `need` makes them:
// an eighth more (less 1/128, which pays for the bitmaps of work_c_ints), so
// that slightly larger graphs find room.  Any later n up to this one uses the
// same arrays, so no kernel may count on the slack of its own n.  A multiple of
// four: supports are read in 16-byte loads.
constexpr long long work_capacity(long long need) {
    return (need + need / 8 - need / 128 + 64) / 4 * 4;
}

// Words of a status bitmap of n vertices, with the one past the end that
// ac6_init may write, up to a cache line.
constexpr long long round_bitmap_words(long long n) { return ((n + 31) / 32 + 2 + 31) / 32 * 32; }

// AC-6 of explicit graphs watches supports from more vertices than this on, with
// late registration at every size (ac6.hip).  From this size on the filters of
// its rounds find room in the list heads, which are made last.
constexpr long long kWatchMinN = 4096;

// Two-sided trimming watches supports from this many vertices on (ac6_two.hip).
constexpr long long kTwoWatchMinN = 4096;
// It keeps two status bitmaps and, behind them, the in-side supports.
constexpr long long two_watch_ints(long long n) { return 2 * round_bitmap_words(n) + n; }

// Ints of the array w.c (Work) for a capacity.
constexpr long long work_c_ints(long long cap) {
    return cap < kTwoWatchMinN ? cap : two_watch_ints(cap);
}

// AC-4's long lists in pieces of whole steps: at most n + m / piece <= 1.5 n pieces,
// for which three arrays of n ints have room (eight bytes each).
constexpr int piece_entries(long long n, long long m, int step) {
    const long long k = n > 0 && m > 0 ? (2 * m + n - 1) / n : 1;
    return k > (1 << 30) ? 1 << 30 : (int)((k + step - 1) / step * step);
}

// Edge positions go up to 2^31 - 1, the end of the last list, so a scan in steps
// of several entries keeps them unsigned: a position plus a step stays below 2^32.
// Entry j of the step at p of a list that ends at e, the last one from there on.
constexpr uint32_t step_index(uint32_t p, int j, int e) {
    return p + (uint32_t)j < (uint32_t)e ? p + (uint32_t)j : (uint32_t)e - 1;
}

// Supports in LDS (watch.h): 16 bits each, for up to this many vertices.
constexpr int kWatchLdsN = 65536;
constexpr int kWatchReads = 4;   // 32-bit reads per lane in flight in a watch pass
// Entries of the support array: n rounded up to whole batches of
// 2 * kWatchReads vertices per lane.
constexpr int watch_padded(int n, int lanes) {
    const int batch = 2 * kWatchReads * lanes;
    return (n + batch - 1) / batch * batch;
}
// Whether an array of `room` entries holds them.  (Not every n up to the room:
// 65,536 vertices are 67,584 entries with 768 lanes.)
constexpr bool watch_fits(long long n, int lanes, int room) {
    return n <= room && watch_padded((int)n, lanes) <= room;
}

}  // namespace trim
