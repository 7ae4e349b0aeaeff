/* The edge chunks' estimates in 8 bytes, run on the host: `steps` blends of `count` nodes, one after the other. */
#include "grem_es_estimate.hip.h"

extern "C" void run_blends(int64_t count, int64_t steps, const uint32_t *h, double *sums, int32_t *lean, uint8_t *widened)
{
    for (int64_t node = 0; node < count; ++node) {
        uint2 word = make_uint2(0u, 0u);
        double2 doubles = make_double2(0.0, 0.0);
        for (int64_t i = 0; i < steps; ++i) {
            const int64_t at = node * steps + i;
            const EsBlended now = es_blend(word, doubles, i > 0, h[2 * at], h[2 * at + 1]);
            if (now.fits) {
                word = now.word;
            } else {
                const size_t place = (size_t)node << 20 | 12345u;
                if (es_is_wide(word) && es_wide_place(word) != place) return;
                word = es_wide_word(place);
                doubles = now.sums;
            }
            const double2 is = es_is_wide(word) ? doubles : es_unpack(word);
            sums[2 * at] = is.x;
            sums[2 * at + 1] = is.y;
            lean[at] = now.lean;
            widened[at] = es_is_wide(word);
        }
    }
}
