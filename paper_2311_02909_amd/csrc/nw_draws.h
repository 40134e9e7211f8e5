// The draws of a node-wise row by one lane (Sec. 4.1.2), shared by the sampling kernels.
#pragma once
#include "bms_device.h"

namespace bms {

// Independent draws (ITS with replacement on the unit weights of a row): s integers in [0, deg), kept sorted
// in c[0..s) by one bubble pass per draw.  Returns the number of distinct values.
template <int S>
__device__ __forceinline__ int32_t replace_draws(uint64_t key, uint32_t deg, int32_t s, uint32_t (&c)[S])
{
#pragma unroll
    for (int j = 0; j < S; ++j) {
        if (j < s) {
            c[j] = bounded32(draw32(key, (uint32_t)j), deg);
#pragma unroll
            for (int q = j; q > 0; --q) {
                const uint32_t lo = min(c[q - 1], c[q]);
                const uint32_t hi = max(c[q - 1], c[q]);
                c[q - 1] = lo;
                c[q] = hi;
            }
        }
    }
    int32_t m = 0;
#pragma unroll
    for (int j = 0; j < S; ++j)
        if (j < s)
            m += (j == 0 || c[j] != c[j - 1]) ? 1 : 0;
    return m;
}

// Draws without replacement, s < deg: draw j is an integer x in [0, deg - j), the index of the pick among the
// positions not chosen so far in ascending order (inverse-transform sampling on the unit weights with the chosen
// entries zeroed).  Stepping x over every chosen position <= x, in ascending order, turns it into the position; the
// list c[0..s) is kept sorted by one bubble pass, which also leaves the row's output in ascending column order.
template <int S>
__device__ __forceinline__ void distinct_draws(uint64_t key, uint32_t deg, int32_t s, uint32_t (&c)[S])
{
#pragma unroll
    for (int j = 0; j < S; ++j) {
        uint32_t x = bounded32(draw32(key, (uint32_t)j), deg - (uint32_t)j);
#pragma unroll
        for (int q = 0; q < j; ++q)
            x += (x >= c[q]) ? 1u : 0u;
        x = j < s ? x : 0xFFFFFFFFu;
        c[j] = x;
#pragma unroll
        for (int q = j; q > 0; --q) {
            const uint32_t lo = min(c[q - 1], c[q]);
            const uint32_t hi = max(c[q - 1], c[q]);
            c[q - 1] = lo;
            c[q] = hi;
        }
    }
}

} // namespace bms
