// The ascending runs in the ids of a large feature fetch (kernels_features.hip): what is decided about them, apart from who
// computes it.  Plain integer code for the device and the host; tests/test_feature_runs.py runs it on the host.
#pragma once

#include <cstdint>

namespace bms {

constexpr int kFetchSamples = 1024;
constexpr int kFetchMostRuns = 512;
constexpr int kFetchTile = 128; // rows per tile of the fetch, on average
constexpr int kFetchLanes = 64;

// place of sample s, s < kFetchSamples, and of the probe between samples s and s + 1: at no fixed distance, so that runs which
// repeat at the samples' distance do not hide.  m >= 64 kFetchSamples.
__host__ __device__ inline int64_t sample_place(int s, int64_t m) { return (int64_t)s * (m - 1) / (kFetchSamples - 1); }
__host__ __device__ inline int64_t probe_place(int s, int64_t m)
{
    const int64_t b = sample_place(s, m), gap = sample_place(s + 1, m) - b;
    uint32_t x = (uint32_t)s * 0x9E3779B9u;
    x ^= x >> 15;
    x *= 0x85EBCA6Bu;
    x ^= x >> 13;
    return b + 1 + (int64_t)((uint64_t)x * (uint64_t)(gap - 1) >> 32);
}

// Two samples of one run have the ids between them in order.  Of ids without an order two thirds of the probes fall outside,
// and of runs shorter than the samples' distance nearly as many: samples alone cannot tell those from minibatches (they
// descend about every second time, or as often as their distance and the runs' length make it).
__host__ __device__ inline bool probe_off(int32_t sample, int32_t probe, int32_t next) { return probe < sample || probe > next; }

// One probe for four samples will do (every sample and probe is a memory line that every workgroup fetches).
constexpr int kFetchProbes = kFetchSamples / 4;
__host__ __device__ inline int probed_sample(int probe) { return probe * 4 + (probe & 3) < kFetchSamples - 2 ? probe * 4 + (probe & 3) : kFetchSamples - 2; }

// descents: of the steps from one sample to the next; probed: of the ascending steps, off: those of them whose probe is outside.  Up
// to an eighth: a minibatch that lies between two samples is missed and costs a probe or two.
__host__ __device__ inline bool runs_likely(int descents, int probed, int off)
{
    return descents > 0 && descents < kFetchMostRuns && off * 8 <= probed;
}
// longest: of the runs, in rows
__host__ __device__ inline bool runs_balanced(int64_t longest, int64_t runs, int64_t m) { return longest <= 4 * (m / runs); }

__host__ __device__ inline int64_t tiles_per_run(int64_t runs, int64_t m)
{
    const int64_t tiles = (m / runs + kFetchTile - 1) / kFetchTile;
    return tiles > 1 ? tiles : 1;
}

// The places of a tile's begin are computed in doubles: a 64-bit division costs a wave as much as 20 multiplications, and a wave
// makes them for every tile.  Products and sums that are rounded still ascend with j, which is all that is asked of them.
__host__ __device__ inline int64_t share_of(int64_t length, int64_t j, double per_tile) { return (int64_t)((double)length * ((double)j * per_tile)); }

// The ids of a tile: those from tile_value(j) on, below tile_value(j + 1), the same in all runs.  Between two samples of run 0, or
// the last one and the run's end, the values are spread evenly.  Samples of a run ascend, whatever the other ids do, so the
// values do too.  per_tile: 1 / tiles, samples_per_row: (kFetchSamples - 1) / (m - 1).
__host__ __device__ inline int64_t tile_value(const int32_t *__restrict__ ids, const int32_t *samples, const int64_t *bounds, int64_t j,
                                              double per_tile, double samples_per_row, int64_t m)
{
    const int64_t last = bounds[1] - 1, p = share_of(last, j, per_tile);
    int s = (int)((double)p * samples_per_row);
    s = s < kFetchSamples - 1 ? s : kFetchSamples - 1;
    s -= sample_place(s, m) > p ? 1 : 0;
    const int64_t p0 = sample_place(s, m), x0 = samples[s];
    int64_t p1 = last, x1;
    if (s + 1 < kFetchSamples && sample_place(s + 1, m) <= last) {
        p1 = sample_place(s + 1, m);
        x1 = samples[s + 1];
    } else {
        x1 = ids[last];
        x1 = x1 < x0 ? x0 : x1;
    }
    const int64_t x = p1 > p0 ? x0 + (int64_t)((float)(x1 - x0) * ((float)(p - p0) / (float)(p1 - p0))) : x0;
    return x < x1 ? x : x1; // (p may lie a row past p1 and the quotient be rounded up)
}

// how far from its share of a run of that length a tile may begin
__host__ __device__ inline int64_t tile_reach(int64_t length) { return length > 16 * 4096 ? length / 16 : 4096; }

// Rows of run r before tile j, j in (0, tiles): the run is searched for the tile's first value in three steps of 64 probes (below(p,
// step, e, v): a bit per x < 64, set if p + x * step < e and ids[p + x * step] < v), exactly in runs of up to 2^18 rows.
// Every step counts set bits at places that only the steps before it choose: whatever order the ids have, a larger value gets
// no smaller a place, and the tiles of a run follow one another without a gap or a row in common.  For the same reason the
// place may be kept to those near the tile's share of the run, which bounds a tile's length.
template <class Below>
__host__ __device__ inline int64_t tile_begin(const int64_t *bounds, int64_t r, int64_t j, double per_tile, int64_t value, Below below)
{
    const int64_t b = bounds[r], e = bounds[r + 1];
    int64_t lo = b, width = e - b;
    for (int level = 0; level < 3 && width > 0; ++level) {
        const int64_t step = (width + kFetchLanes - 1) / kFetchLanes;
        const int64_t end = lo + width;
        const int64_t count = __builtin_popcountll(below(lo, step, end, value));
        if (level == 2 || step == 1) {
            lo = lo + count * step < end ? lo + count * step : end;
            break;
        }
        if (count == 0)
            break;
        lo += (count - 1) * step;
        width = end - lo < step ? end - lo : step;
    }
    const int64_t share = b + share_of(e - b, j, per_tile);
    const int64_t most = tile_reach(e - b);
    lo = lo < share - most ? share - most : lo;
    lo = lo > share + most ? share + most : lo;
    return lo < b ? b : lo > e ? e : lo;
}

} // namespace bms
