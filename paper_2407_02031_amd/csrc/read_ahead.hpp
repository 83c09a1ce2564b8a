// What launches behind this one will read (their weights), brought into the last-level cache by workgroups of 256 threads behind
// the launch's own (in the chain by its own workgroups, when they are done): each reads LOADS * 4 KB of the ranges, taken as one string of bytes, all of it in flight at once,
// and uses nothing.  (Loads with the non-temporal hint are not kept in that cache.)
//
// A deep stack's weights do not stay in the last-level cache from block to block, and a projection of one round of tiles has
// nothing to hide HBM's latency behind (ten blocks of 1280 channels, own weights / one block's weights for all ten: 32 x 32
// tokens 2699 / 2446 us, 26 x 38 tokens 1734 / 1475).  Attention and LayerNorm hardly use HBM.  What bounds it: HBM and the launch
// it rides in.  ff2 of 2048 x 1280 x 5120 + 64 51.5 -> 39.8 us and of 988 rows 34 -> 28, ff1 of 988 rows 36 -> 30, q, k, v 48 -> 44;
// self-attention over 1024 tokens that reads 36 MB 21.3 -> 25, LayerNorm that reads 8 MB 5.2 -> 6.6.
#pragma once
#include "common.hpp"

namespace sd {

template <int LOADS>
__device__ __forceinline__ void read_ahead(const ReadRanges& ra, int wg, int tid) {
    constexpr uint32_t STEP = READ_AHEAD_STEP, UNIT = LOADS * STEP;
    // lane i holds range i and where it starts in the string
    const int lane = tid & 63;
    const bool has = lane < ra.n;
    const uint64_t base = has ? reinterpret_cast<uint64_t>(ra.p[lane]) : 0;
    const uint32_t size = has ? ra.bytes[lane] : 0u, start = has ? ra.start[lane] : 0u;
    const uint32_t lo = (uint32_t)wg * UNIT, hi = lo + UNIT;
    uint64_t mine = __builtin_amdgcn_ballot_w64(has && start < hi && start + size > lo);
#pragma unroll 1
    for (; mine; mine &= mine - 1) {
        const int i = __builtin_ctzll(mine);
        const uint32_t rs = (uint32_t)__builtin_amdgcn_readlane((int)start, i), rn = (uint32_t)__builtin_amdgcn_readlane((int)size, i);
        const char* const p = reinterpret_cast<const char*>(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(base >> 32), i) << 32) |
                                                            (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)base, i));
        const uint32_t at = lo > rs ? lo - rs : 0u, end = hi - rs < rn ? hi - rs : rn;
        u32x4 v[LOADS];
#pragma unroll
        for (uint32_t u = 0; u < LOADS; ++u) {
            const uint32_t off = at + u * STEP + (uint32_t)tid * 16u;
            v[u] = u32x4{0u, 0u, 0u, 0u};
            if (off < end) v[u] = *(const __attribute__((address_space(1))) u32x4*)(p + off);    // sizes are multiples of 16
        }
#pragma unroll
        for (uint32_t u = 0; u < LOADS; ++u) asm volatile("" ::"v"(v[u]));
    }
}

}  // namespace sd
