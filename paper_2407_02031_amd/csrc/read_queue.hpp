// Device memory that coming launches will read (a stack's weights), and which launch ahead of them brings what part of it into
// the last-level cache.  Host code; the device side is read_ahead.hpp.
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <algorithm>
#include <vector>

namespace sd {

constexpr uint32_t READ_AHEAD_STEP = 4096;   // bytes of one load of a workgroup (256 threads)

// The part that one launch reads, with `wgs` workgroups behind its own.
struct ReadRanges {
    static constexpr int MAX = 24;
    const void* p[MAX];
    uint32_t bytes[MAX], start[MAX];   // multiples of 16; where each begins in the string of all
    int32_t n, wgs;
};
struct NoRanges {};                    // the argument of kernels that read none

// The queue the parts come from, in order of use.
struct ReadAhead {
    // No part begins or ends further ahead of the launches than this.  It has to reach across both feed-forward projections, because
    // nothing reads between them: 39 MB at 1280 channels without adapters, 10 at 640; what lies beyond is driven out again before its
    // turn.  One number for all: swept at 26 x 38 tokens, one sample, ten blocks of 1280 channels, 62 MB a block (us per stack: without 1806,
    // 32 MB 1662, 40 MB 1569, 44 MB 1627, 64 MB 1645, 96 MB 1672, no limit 1647).  With adapters of rank 64 and the next block's text weights
    // in ff2 (32 x 32 tokens) the two launches read 52 MB, of which the last 12 come from HBM.
    static constexpr uint64_t LEAD = 40ull << 20;
    struct Range { const char* p; uint64_t bytes; };
    std::vector<Range> ranges;
    std::vector<uint64_t> marks;       // where in the string of all ranges those of each launch end
    size_t at = 0, launch = 0;         // first range not handed out whole; launches so far
    uint64_t at_start = 0, done = 0, total = 0;

    void add(const void* q, size_t size) {
        size &= ~(size_t)15;
        if (!q || size == 0) return;
        ranges.push_back({static_cast<const char*>(q), size});
        total += size;
    }
    void mark() { marks.push_back(total); }
    // a launch has been enqueued: its own ranges need no reading any more
    void launched() {
        if (launch < marks.size()) done = std::max(done, marks[launch]);
        ++launch;
    }
    // the next `budget` bytes, as far as `room` workgroups of `loads` loads go
    ReadRanges take(uint64_t budget, long room, int loads) {
        ReadRanges r;
        r.n = r.wgs = 0;
        const uint64_t unit = (uint64_t)loads * READ_AHEAD_STEP;
        const uint64_t to = (launch && !marks.empty() ? marks[std::min(launch, marks.size()) - 1] : 0) + LEAD;
        uint64_t most = room < 16 ? 0 : std::min(budget, room * unit);
        most = std::min(most, to > done ? to - done : 0) & ~(uint64_t)15;
        uint64_t got = 0;
        while (got < most && r.n < ReadRanges::MAX && at < ranges.size()) {
            const Range& g = ranges[at];
            if (at_start + g.bytes <= done) {
                at_start += g.bytes;
                ++at;
                continue;
            }
            const uint64_t from = done - at_start, n = std::min(g.bytes - from, most - got);
            r.p[r.n] = g.p + from;
            r.bytes[r.n] = (uint32_t)n;
            r.start[r.n++] = (uint32_t)got;
            got += n;
            done += n;
        }
        r.wgs = (int32_t)((got + unit - 1) / unit);
        return r;
    }
};

}  // namespace sd
