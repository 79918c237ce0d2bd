// segment_search.hpp -- the index arithmetic of the wave-wide search of
// segment offsets (wave_lower_bounds in scan_kernel.hpp).  No HIP dependency:
// the functions are constexpr, so they run on the device and in a CPU test
// that counts every index probed.
#pragma once

#include <cstdint>

namespace lscan {

// The first index k with off[k] >= v lies in [lo, hi]; off[hi] is not below v
// or hi is the number of offsets.  Each round probes up to 64 indices of
// [lo, hi), `step` apart, and cuts the range by 65.  Two such searches share
// one loop, so a search that has ended (lo == hi) takes further rounds: it
// probes nothing and stays as it is.
struct OffsetRange {
    int64_t lo, hi;
};

constexpr bool range_open(const OffsetRange& r) { return r.lo < r.hi; }

// 1 once at most 65 indices are left, 0 for a search that has ended
constexpr int64_t probe_step(const OffsetRange& r) { return (r.hi - r.lo + 64) / 65; }

constexpr int64_t probe_index(const OffsetRange& r, int64_t step, int lane) { return r.lo + (lane + 1) * step - 1; }

// Whether index p of a round is read: only then does it lie in [lo, hi).
constexpr bool probe_reads(const OffsetRange& r, int64_t p) { return r.lo <= p && p < r.hi; }

// The range after a round in which `below` of the probes read were below v.
// Offsets that decrease somewhere leave it inside the old one all the same.
constexpr OffsetRange narrowed(const OffsetRange& r, int64_t step, int64_t below)
{
    if (!range_open(r)) return r;
    const int64_t first = r.lo + below * step;
    const int64_t end = first + step - 1;  // the first probe not below, if there is one
    if (below < 64 && end < r.hi) return OffsetRange{first, end};
    return OffsetRange{first < r.hi ? first : r.hi, r.hi};
}

}  // namespace lscan
