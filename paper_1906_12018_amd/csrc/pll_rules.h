// The rules that choose the lanes of a query call, on sizes alone (plain C++:
// the functions run on the host as well as in the library).
#pragma once

#include <stdint.h>

namespace pll {

// What the rules look at: n vertices, `entries` label entries (the mean of
// both sides of a directed index), the longest label, bit-parallel roots.
struct LabelShape {
    uint64_t n, entries, longest, roots;
};

constexpr uint64_t label_mean(const LabelShape& s) { return s.n ? s.entries / s.n : 0; }

// Labels of like lengths: none is eight times the mean.  (R-MAT: 12 to 16
// times, half of its pairs meeting an isolated vertex; Barabasi-Albert, trees
// and tori: 2 to 6 times.)
constexpr bool labels_even(const LabelShape& s) { return s.longest * s.n < 8 * s.entries; }

// Lanes per pair of a large call: the window of a group (4 entries per lane)
// should hold about one average label.  From a mean of 32 entries on a whole
// wave per pair (R-MAT indexes of 2^14..2^20 vertices, means of 44..241: the
// fastest at every size).  With bit-parallel roots every pair has the bound
// to compute, for which a wave has more lanes than roots, and groups stay
// ahead longer, 1,000,000 pairs with 16 and 64 lanes: Barabasi-Albert, means
// of 34 to 70: 187 and 464 us, 241 and 490, 305 and 528; a torus, 63: 217 and
// 419.  In R-MAT indexes, whose few long labels decide a group's time, they
// do so up to a mean of 48 (38: 254 and 307; 45: 287 and 315; 50: 320 and
// 302; 58: 357 and 316), and with 32 roots or more, whose sets keep a wave's
// lanes busy, not at all (32, 64 roots: 379 and 321; 43: 453 and 329).
// From 16 roots on 8 lanes share them (mean 17, 16 roots: 157 us, 172 with 4
// lanes; mean 4.8, 64 roots: 234 and 391).
constexpr uint32_t query_lanes(const LabelShape& s) {
    const uint64_t mean = label_mean(s);
    if (mean >= (s.roots ? 64u : 32u)) return 64;
    if (mean >= 32 && !labels_even(s) && (mean >= 48 || s.roots >= 32)) return 64;
    uint32_t g = s.roots >= 16 ? 8 : 4;
    while (g < 32 && 4ull * g < mean) g *= 2;
    return g;
}

// Calls of up to this many pairs take a wave per pair whatever the mean label
// (when the index leaves the lanes open): they do not fill the device, so the
// longest pair's chain of windows decides.  Mean labels of 4 to 43 entries,
// 8,000 pairs: 8.4-9.0 us, 14-44 us with groups; 30,000 pairs: 14-26 us
// against 18-30; from 100,000 pairs on the groups win.  Short even labels
// with fewer than 32 roots on 32,768 vertices or more cross over sooner: a
// tree of 200,000, 4 roots, 24,576, 28,672 and 32,768 pairs 20.1, 23.4 and
// 26.5 us, 20.5, 21.4 and 21.5 with groups.
constexpr uint64_t query_small_call(const LabelShape& s) {
    const bool sooner = s.roots && s.roots < 32 && s.n >= 32768 && label_mean(s) < 32 && labels_even(s);
    return sooner ? 24576 : 32768;
}

}  // namespace pll
