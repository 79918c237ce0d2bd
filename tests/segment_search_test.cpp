// The wave-wide search of segment offsets, lane by lane on the CPU: every
// index that a lane reads has to lie inside the offsets, and the two results
// have to be the first indices not below the two values.
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

#include "segment_search.hpp"

using namespace lscan;

static long failures = 0;
static void fail(const char* what, int64_t S, int64_t a, int64_t b)
{
    if (++failures <= 20) std::printf("FAIL %s: S=%lld a=%lld b=%lld\n", what, (long long)S, (long long)a, (long long)b);
}

// The kernel's loop with at(k) for off[k]; the indices are checked before they are used.
template <class At>
static void search(int64_t S, int64_t v0, int64_t v1, const At& at, int64_t& k0, int64_t& k1)
{
    OffsetRange r[2] = {{0, S}, {0, S}};
    const int64_t v[2] = {v0, v1};
    for (int round = 0; range_open(r[0]) || range_open(r[1]); ++round) {
        if (round > 64) return fail("does not end", S, v0, v1);
        for (int q = 0; q < 2; ++q) {
            const int64_t step = probe_step(r[q]);
            int64_t below = 0;
            for (int lane = 0; lane < 64; ++lane) {
                const int64_t p = probe_index(r[q], step, lane);
                if (!probe_reads(r[q], p)) continue;
                if (p < 0 || p >= S) {
                    fail("reads outside the offsets", S, p, round);
                    continue;
                }
                below += at(p) < v[q] ? 1 : 0;
            }
            const OffsetRange n = narrowed(r[q], step, below);
            if (n.lo < r[q].lo || n.hi > r[q].hi || n.lo > n.hi) fail("range grows", S, n.lo, n.hi);
            r[q] = n;
        }
    }
    k0 = r[0].lo;
    k1 = r[1].lo;
}

// Sorted offsets of which m0 lie below the first value and m1 below the second.
static void sorted_case(int64_t S, int64_t m0, int64_t m1)
{
    int64_t k0 = -1, k1 = -1;
    search(S, 1, 2, [&](int64_t k) { return k < m0 ? 0 : k < m1 ? 1 : 2; }, k0, k1);
    if (k0 != m0 || k1 != m1) fail("wrong bounds", S, k0 - m0, k1 - m1);
}

int main()
{
    // the first block (nothing below its start), with every number of offsets in it
    std::vector<int64_t> counts;
    for (int64_t S = 0; S <= 700; ++S) counts.push_back(S);
    for (int64_t S = 4150; S <= 4360; ++S) counts.push_back(S);  // around two full rounds
    for (int64_t S = 701; S <= 5000; S += 53) counts.push_back(S);
    for (int64_t S : counts)
        for (int64_t m = 0; m <= S; ++m) sorted_case(S, 0, m);
    // later blocks, and counts of many rounds
    std::mt19937_64 g(1604);
    for (int i = 0; i < 200000; ++i) {
        const int64_t S = int64_t(g() % (int64_t(1) << (1 + g() % 24)));
        int64_t a = int64_t(g() % uint64_t(S + 1)), b = int64_t(g() % uint64_t(S + 1));
        if (a > b) std::swap(a, b);
        sorted_case(S, a, b);
        sorted_case(S, a, a);
        sorted_case(S, a, S);
    }
    // offsets in no order: some index in [0, S], and no other read
    for (int i = 0; i < 60000; ++i) {
        const int64_t S = int64_t(g() % (i % 2 ? 300 : 5000));
        std::vector<int64_t> off(static_cast<size_t>(S));
        for (auto& o : off) o = int64_t(g() % 64) - 16;
        int64_t k0 = -1, k1 = -1;
        search(S, int64_t(g() % 80) - 20, int64_t(g() % 80) - 20, [&](int64_t k) { return off[size_t(k)]; }, k0, k1);
        if (k0 < 0 || k0 > S || k1 < 0 || k1 > S) fail("index outside [0, S]", S, k0, k1);
    }
    if (failures) {
        std::printf("%ld failures\n", failures);
        return 1;
    }
    std::printf("all checks passed\n");
    return 0;
}
