// How a look-up launch of the two-phase route (k_tp_lookup) deals column blocks out to workgroups: plain arithmetic, the same on the
// host, where a test runs it over blocks of very unequal sizes (ids in order of degree: the first blocks hold most
// entries).  All sizes are in groups of eight tuples; every share is an equal part of one block's.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace grem {

struct LookupShares {
    uint32_t few, many;    // a chunk's launch: workgroups of a block whose shares would be short, and at most
    uint32_t per;          // a sweep over all blocks (not 0): most groups of a share
};

// A chunk's launch has `many` workgroups per block; a block's shares: each workgroup copies the block's labels (64 KB) first, so short
// shares are few (13.9M vertices in chunks of 2^17 and k = 32, 512 | 256 workgroups a chunk: 8.75 | 8.33 ms), long ones many (in chunks of
// 2^20 by degree, k = 16, seeded: 9.8 | 13.6 ms; all the same where a block has 235,000 groups for 16 or 32, but 28 shares of it, not whole eights
// and so on other XCDs than its neighbours', cost the first call on 111M vertices 50.2 -> 51.6 ms).
constexpr uint32_t kLookupLong = 16384;
__host__ __device__ inline uint32_t lookup_chunk_shares(uint32_t groups, const LookupShares &d) {
    const uint32_t wanted = d.few % 8u == 0u ? groups / kLookupLong & ~7u : groups / kLookupLong;
    return wanted < d.few ? d.few : wanted < d.many ? wanted : d.many;
}

// A sweep's workgroups in the order of the blocks: block j, whose groups are [start, end) of all, has those from lookup_first(start, j)
// up to the next block's first one: no share is longer than `per`, whatever the blocks' sizes, and there are total / per + blocks of them.
__host__ __device__ inline uint32_t lookup_first(uint32_t start, uint32_t j, const LookupShares &d) { return start / d.per + j; }
__host__ __device__ inline uint32_t lookup_sweep_shares(uint32_t start, uint32_t end, const LookupShares &d) { return end / d.per - start / d.per + 1u; }
inline uint32_t lookup_sweep_grid(uint64_t groups, uint32_t blocks, const LookupShares &d) { return (uint32_t)(groups / d.per) + blocks; }

}  // namespace grem
