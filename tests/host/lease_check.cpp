// Leases of whole solves: however the workgroups of all leases held are placed,
// each finds a place on its XCD. Placement is as unkind as the hardware can
// be: leases are dispatched in any interleaving, each launch's workgroups to the
// XCDs in turn from any first XCD, and a workgroup that shares a CU takes an
// empty one while there is one.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "swgn_lease.h"

using namespace swgn::rt;

static void fail(const char* what, int a, int b) {
    std::printf("%s (%d, %d)\n", what, a, b);
    std::exit(1);
}

struct Lease {
    bool alone;
    int n;
};

int main() {
    std::mt19937 rng(7);
    auto pick = [&](int lo, int hi) { return std::uniform_int_distribution<int>(lo, hi)(rng); };
    const int cus = 256, per = cus / kXcds;
    long placed = 0;
    int refused = 0;
    for (int trial = 0; trial < 2000; ++trial) {
        PcgHeld held;
        std::vector<Lease> leases;
        const int only = pick(0, 2);                 // one kind only, or both
        for (int k = pick(1, 40); k > 0; --k) {
            if (!leases.empty() && pick(0, 3) == 0) {
                const size_t q = (size_t)pick(0, (int)leases.size() - 1);
                pcg_give(held, leases[q].alone, leases[q].n);
                leases.erase(leases.begin() + (long)q);
                continue;
            }
            const bool alone = only == 0 ? false : (only == 1 ? true : pick(0, 1) == 1);
            const int most = pick(2, pick(2, cus)), all = most + pick(0, 300);
            const int n = pcg_take(held, alone, cus, most, all);
            if (n == 0) { ++refused; continue; }
            if (n < most || n % kXcds != 0) fail("a lease below its largest solve, or not whole XCDs", n, most);
            leases.push_back({alone, n});
        }
        int pair = 0, alone = 0;
        for (const Lease& l : leases) (l.alone ? alone : pair) += l.n;
        if (pair != held.pair || alone != held.alone) fail("leases and what is held differ", pair, held.pair);
        // place them: load[x][c] halves of CU c of XCD x
        std::vector<std::vector<int>> load(kXcds, std::vector<int>((size_t)per, 0));
        std::vector<int> left, at;
        for (const Lease& l : leases) {
            left.push_back(l.n);
            at.push_back(pick(0, kXcds - 1));
        }
        for (;;) {
            std::vector<size_t> open;
            for (size_t q = 0; q < left.size(); ++q)
                if (left[q] > 0) open.push_back(q);
            if (open.empty()) break;
            const size_t q = open[(size_t)pick(0, (int)open.size() - 1)];
            std::vector<int>& x = load[(size_t)(at[q] % kXcds)];
            int c = -1;
            for (int v = 0; v < per && c < 0; ++v)
                if (x[(size_t)v] == 0) c = v;
            for (int v = 0; v < per && c < 0 && !leases[q].alone; ++v)
                if (x[(size_t)v] == 1) c = v;
            if (c < 0) fail("a leased workgroup finds no place", (int)held.pair, (int)held.alone);
            x[(size_t)c] += leases[q].alone ? 2 : 1;
            --left[q];
            ++at[q];
            ++placed;
        }
    }
    if (placed < 100000 || refused < 1000) fail("the trials do not fill the device", (int)placed, refused);
    // an idle device gives a batch everything, and then nothing more to anyone
    PcgHeld h;
    if (pcg_take(h, true, cus, 65, 520) != cus || pcg_take(h, false, cus, 2, 2) != 0) fail("whole device", h.alone, h.pair);
    pcg_give(h, true, cus);
    if (h.alone != 0 || h.pair != 0) fail("given back", h.alone, h.pair);
    // streams that share CUs: two full rounds of them
    if (pcg_take(h, false, cus, 56, cus) != cus || pcg_take(h, false, cus, 56, cus) != cus) fail("pairs", h.pair, 0);
    if (pcg_take(h, false, cus, 2, 8) != 0) fail("beyond pairs", h.pair, 0);
    std::printf("placed %ld, refused %d\nok\n", placed, refused);
    return 0;
}
