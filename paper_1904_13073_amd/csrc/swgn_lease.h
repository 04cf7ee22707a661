// Which whole linear solves (pcg.hip) of a process may run on a device at once.
//
// A solve's workgroups wait for each other, so every one of them must get a
// place whatever is already placed. A workgroup is of one of two kinds: of the
// first a CU holds two, one of the second takes a CU for itself. Workgroups
// of the first kind may be spread one per CU, which leaves no CU for the
// second. So while any of the second are leased, each workgroup counts as
// a CU; only where all are of the first kind do two count as one. And the
// workgroups of a launch go to the XCDs in turn, whatever their load, so a
// launch of n puts up to ceil(n / 8) on one XCD: leases are multiples of the
// number of XCDs.
#pragma once

#include <algorithm>

namespace swgn {
namespace rt {

constexpr int kXcds = 8;

// workgroups leased on a device
struct PcgHeld {
    int pair = 0, alone = 0;                  // two per CU, one per CU
};

// how many more of a kind are sure of a place
inline int pcg_room(const PcgHeld& h, bool alone, int cus) {
    const int cap = alone || h.alone > 0 ? cus : 2 * cus;
    return std::max(0, (cap - h.pair - h.alone) / kXcds * kXcds);
}

// Leases what launches of `all` workgroups in all can use, at least `most` (the
// largest solve), or nothing: the number leased.
inline int pcg_take(PcgHeld& h, bool alone, int cus, int most, int all) {
    const int want = (all + kXcds - 1) / kXcds * kXcds;
    const int n = std::min(want, pcg_room(h, alone, cus));
    if (n < most) return 0;
    (alone ? h.alone : h.pair) += n;
    return n;
}

inline void pcg_give(PcgHeld& h, bool alone, int n) { (alone ? h.alone : h.pair) -= n; }

}  // namespace rt
}  // namespace swgn
