/* The look-up launches' division of column blocks into shares, on the host. */
#include <vector>

#include "grem_lookup_shares.hip.h"

using namespace grem;

/* A sweep over blocks that start at start[0..blocks]: deals every workgroup its share as the kernel does and returns the longest
 * share, or -1 if a group is not dealt exactly once. */
extern "C" int64_t longest_sweep_share(const uint32_t *start, uint32_t blocks, uint32_t per)
{
    const LookupShares d{1u, 1u, per};
    const uint32_t grid = lookup_sweep_grid(start[blocks], blocks, d);
    int64_t longest = 0;
    uint64_t at = 0;                                     /* dealt so far */
    for (uint32_t id = 0, j = 0; id < grid; ++id) {
        while (j + 1 < blocks && lookup_first(start[j + 1], j + 1, d) <= id) ++j;
        const uint32_t s = id - lookup_first(start[j], j, d), shares = lookup_sweep_shares(start[j], start[j + 1], d);
        if (s >= shares) continue;
        const uint64_t groups = start[j + 1] - start[j], g0 = groups * s / shares, g1 = groups * (s + 1) / shares;
        if (start[j] + g0 != at) return -1;
        at += g1 - g0;
        if ((int64_t)(g1 - g0) > longest) longest = (int64_t)(g1 - g0);
    }
    return at == start[blocks] ? longest : -1;
}

extern "C" uint32_t chunk_shares(uint32_t groups, uint32_t few, uint32_t many) { return lookup_chunk_shares(groups, LookupShares{few, many, 0u}); }
