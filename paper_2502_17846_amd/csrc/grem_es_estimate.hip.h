// A node's two estimates (Alg. 1's nbr_counts) in 8 bytes, and their blend with a chunk's fresh counts: plain arithmetic, the
// same on the host, where tests run it against doubles.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstddef>
#include <cstdint>

// Both counts as whole numbers of 29 bits and, in the six bits above them, how many times they have
// been halved, which is all of the doubles' value while no bit of it is lost.  Once one does not fit (a node has 29 edge ends or
// more by then) the two are doubles in an array of their own and the 58 bits say where.
constexpr uint32_t kPackBits = 29, kPackMask = (1u << kPackBits) - 1u, kPackWide = 7u << kPackBits;
__host__ __device__ __forceinline__ bool es_is_wide(uint2 word) { return word.y >= kPackWide; }
__host__ __device__ __forceinline__ size_t es_wide_place(uint2 word) { return (word.x & kPackMask) | (size_t)(word.y & kPackMask) << kPackBits; }
__host__ __device__ __forceinline__ uint2 es_wide_word(size_t place) { return make_uint2((uint32_t)place & kPackMask, (uint32_t)(place >> kPackBits) | kPackWide); }
__host__ __device__ __forceinline__ uint32_t es_halved(uint2 word) { return word.x >> kPackBits | (word.y >> kPackBits) << 3; }
__host__ __device__ __forceinline__ uint2 es_pack(uint32_t x, uint32_t y, uint32_t halved)
{
    return make_uint2(x | halved << kPackBits, y | (halved >> 3) << kPackBits);
}
__host__ __device__ __forceinline__ double2 es_unpack(uint2 word)
{
    const int halved = (int)es_halved(word);
    return make_double2(ldexp((double)(word.x & kPackMask), -halved), ldexp((double)(word.y & kPackMask), -halved));
}

struct EsBlended {
    bool fits;        // in 8 bytes: `word`; otherwise `sums`
    uint2 word;
    double2 sums;
    int lean;         // +1 where side 1 holds more, -1 where side 0 does, 0: neither
};
// word, doubles: the stored estimate (doubles: of a wide word), zero for a node that is not blended (or a wide word and zeros, where
// all estimates are doubles).  Where it grows out of 29 bits, the sums are rounded on their way into the doubles as the doubles' own sums would be, and it is the doubles that are compared.
__host__ __device__ __forceinline__ EsBlended es_blend(uint2 word, double2 doubles, bool blend, uint32_t h0, uint32_t h1)
{
    EsBlended r{};
    if (es_is_wide(word)) {
        const double share = blend ? 0.5 : 1.0;
        r.sums = make_double2((doubles.x + (double)h0) * share, (doubles.y + (double)h1) * share);
    } else {
        const uint32_t b = es_halved(word), halved = b + (blend ? 1u : 0u);
        const uint32_t x0 = word.x & kPackMask, y0 = word.y & kPackMask;
        if (b < kPackBits && ((h0 | h1) >> (kPackBits - b)) == 0u) {
            const uint32_t x = x0 + (h0 << b), y = y0 + (h1 << b);
            if (((x | y) >> kPackBits) == 0u) {
                r.fits = true;
                r.word = es_pack(x, y, halved);
                r.lean = (y > x) - (x > y);
                return r;
            }
        }
        r.sums = make_double2(ldexp((double)(x0 + ((uint64_t)h0 << b)), -(int)halved), ldexp((double)(y0 + ((uint64_t)h1 << b)), -(int)halved));
    }
    r.lean = (r.sums.y > r.sums.x) - (r.sums.x > r.sums.y);
    return r;
}
