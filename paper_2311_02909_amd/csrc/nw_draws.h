// The draws of a node-wise row by one lane (Sec. 4.1.2), shared by the sampling kernels.
#pragma once
#include "bms_device.h"

namespace bms {

__device__ __forceinline__ uint32_t median(uint32_t x, uint32_t y, uint32_t z) // one instruction
{
    return max(min(x, y), min(max(x, y), z));
}

// Independent draws (ITS with replacement on the unit weights of a row): s integers in [0, deg), kept sorted
// in c[0..s): x goes between the values below and above it, and those above move up, which is the median of x, a place's value and
// the one before it.  Returns the number of distinct values.
template <int S>
__device__ __forceinline__ int32_t replace_draws(uint64_t key, uint32_t deg, int32_t s, uint32_t (&c)[S])
{
#pragma unroll
    for (int j = 0; j < S; ++j) {
        if (j < s) {
            const uint32_t x = bounded32(draw32(key, (uint32_t)j), deg);
            c[j] = j ? max(c[j - 1], x) : x;
#pragma unroll
            for (int q = j - 1; q > 0; --q)
                c[q] = median(c[q - 1], x, c[q]);
            if (j)
                c[0] = min(c[0], x);
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
// entries zeroed).  Stepping x over every chosen position <= x, in ascending order, turns it into the position, that is x + t
// where t positions are stepped over: those with position - place <= x (unchosen positions before them, which never decrease
// along the list).  So the list c[0..s), sorted, becomes in place q the median of c[q - 1], x + q and c[q]: c[q] as long as
// it is stepped over, x + t in place t, and the one before it after that.  No chain through the list: 2 instructions per
// place and draw, where a pass of steps and one of exchanges took 4.
// First hop of one minibatch of 1024 seeds, fanout 15 (one compute unit, where the draws are a fifth of the time): 32.8 -> 30.9 us.
template <int S>
__device__ __forceinline__ void distinct_draws(uint64_t key, uint32_t deg, int32_t s, uint32_t (&c)[S])
{
#pragma unroll
    for (int j = 0; j < S; ++j) {
        if (j < s) { // the same for all lanes
            const uint32_t x = bounded32(draw32(key, (uint32_t)j), deg - (uint32_t)j);
            c[j] = j ? max(c[j - 1], x + (uint32_t)j) : x;
#pragma unroll
            for (int q = j - 1; q > 0; --q)
                c[q] = median(c[q - 1], x + (uint32_t)q, c[q]);
            if (j)
                c[0] = min(c[0], x);
        }
    }
}

// Draws without replacement by one wave, s < deg, s <= 64 K.  The sorted positions lie across the lanes (position t in
// lane t % 64 of register t / 64), kept as e_t = position_t - t: the number of unchosen positions before it, which never
// decreases with t.  A draw x steps over the c positions with e_t <= x and becomes position c, with e_c = x; those after it
// move up by one place, which lowers their e by one.  All draws' x are computed at once, one per lane and register.
// On return e[q] is the position of place 64 q + lane (places >= s: undefined).
template <int K>
__device__ __forceinline__ void wave_distinct_draws(uint64_t key, uint32_t deg, int32_t s, int lane, uint32_t (&e)[K])
{
    uint32_t x_of[K];
#pragma unroll
    for (int q = 0; q < K; ++q) {
        const uint32_t j = (uint32_t)(64 * q + lane);
        x_of[q] = bounded32(draw32(key, j), deg - j); // draws j >= s are never used
        e[q] = 0xFFFFFFFFu; // no position: above every x, also 64 K places lower
    }
#pragma unroll
    for (int qj = 0; qj < K; ++qj) {
        const int32_t jn = min(64, s - 64 * qj);
        for (int32_t j = 0; j < jn; ++j) {
            const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)x_of[qj], j);
            int c = 0;
#pragma unroll
            for (int q = 0; q <= qj; ++q)
                c += __popcll(__ballot(e[q] <= x));
#pragma unroll
            for (int q = qj; q >= 0; --q) {
                const int carry = q ? __builtin_amdgcn_readlane((int)e[q - 1 >= 0 ? q - 1 : 0], kWave - 1) : 0;
                const uint32_t up = (uint32_t)__builtin_amdgcn_update_dpp(carry, (int)e[q], 0x138 /* wave_shr:1 */, 0xF, 0xF, false) - 1u;
                const int t = 64 * q + lane;
                e[q] = t > c ? up : t == c ? x : e[q];
            }
        }
    }
#pragma unroll
    for (int q = 0; q < K; ++q)
        e[q] += (uint32_t)(64 * q + lane);
}

// Independent draws by one wave, s <= 64: sorted across the lanes, lane 0 .. m - 1 of the result hold the distinct
// positions in ascending order.  Returns m.
__device__ __forceinline__ int32_t wave_replace_draws64(uint64_t key, uint32_t deg, int32_t s, int lane, uint32_t &pos)
{
    uint32_t v = lane < s ? bounded32(draw32(key, (uint32_t)lane), deg) : 0xFFFFFFFFu;
    v = wave_sort_u32(v, lane);
    const uint32_t prev = __shfl_up(v, 1, kWave);
    const bool head = lane < s && (lane == 0 || v != prev);
    const uint64_t heads = __ballot(head);
    // lane x takes the value of the (x + 1)-th head
    const int at = __popcll(heads & ((1ull << lane) - 1ull)); // heads before this lane
    pos = (uint32_t)__builtin_amdgcn_ds_permute((head ? at : kWave - 1) * 4, (int)v);
    return __popcll(heads);
}

} // namespace bms
