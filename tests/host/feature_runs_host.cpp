// Host replay of the runs and tiles of a large feature fetch, over the code of csrc/feature_runs.h: what a workgroup of
// feature_fetch_kernel finds, and which rows its tiles are.  Built and loaded by tests/test_feature_runs.py.
#define __host__
#define __device__
#include "feature_runs.h"

#include <algorithm>
#include <cstdlib>
#include <vector>

using namespace bms;

namespace {

std::vector<int64_t> find_runs(const int32_t *ids, int64_t m)
{
    const std::vector<int64_t> none{0, m};
    int descents = 0, probed = 0, off = 0;
    auto sample = [&](int s) { return ids[sample_place(s, m)]; };
    for (int s = 0; s + 1 < kFetchSamples; ++s)
        descents += sample(s + 1) < sample(s) ? 1 : 0;
    for (int x = 0; x < kFetchProbes; ++x) {
        const int s = probed_sample(x);
        if (sample(s) > sample(s + 1))
            continue;
        ++probed;
        off += probe_off(sample(s), ids[probe_place(s, m)], sample(s + 1)) ? 1 : 0;
    }
    if (!runs_likely(descents, probed, off))
        return none;
    std::vector<int64_t> bounds{0};
    for (int s = 0; s + 1 < kFetchSamples; ++s) {
        int64_t lo = sample_place(s, m), hi = sample_place(s + 1, m);
        const int32_t x = ids[lo];
        if (ids[hi] >= x)
            continue;
        while (hi - lo > 1) {
            const int64_t mid = (lo + hi) >> 1;
            (ids[mid] < x ? hi : lo) = mid;
        }
        bounds.push_back(hi);
    }
    bounds.push_back(m);
    int64_t longest = 0;
    const int64_t runs = (int64_t)bounds.size() - 1;
    for (int64_t r = 0; r < runs; ++r)
        longest = std::max(longest, (bounds[r + 1] - bounds[r]) / kFetchTile * kFetchTile);
    return runs_balanced(longest, runs, m) ? bounds : none;
}

} // namespace

// longest tile, in rows; apart: largest distance between the first ids of tile j of a run and of run 0.  Returns the number of
// runs, or -1 if the tiles of a run do not follow one another.
extern "C" int64_t replay(const int32_t *ids, int64_t m, int64_t *longest, int64_t *apart)
{
    const std::vector<int64_t> bounds = find_runs(ids, m);
    const int64_t runs = (int64_t)bounds.size() - 1, tiles = tiles_per_run(runs, m);
    const double per_tile = 1.0 / (double)tiles, samples_per_row = (double)(kFetchSamples - 1) / (double)(m - 1);
    int32_t samples[kFetchSamples];
    for (int s = 0; s < kFetchSamples; ++s)
        samples[s] = ids[sample_place(s, m)];
    auto below = [&](int64_t p, int64_t step, int64_t e, int64_t v) {
        uint64_t bits = 0;
        for (int x = 0; x < kFetchLanes; ++x)
            if (p + x * step < e && ids[p + x * step] < v)
                bits |= 1ULL << x;
        return bits;
    };
    auto begin = [&](int64_t r, int64_t j) -> int64_t {
        if (runs == 1)
            return std::min<int64_t>(j * kFetchTile, m);
        if (j == 0 || j == tiles)
            return bounds[r + (j ? 1 : 0)];
        return tile_begin(bounds.data(), r, j, per_tile, tile_value(ids, samples, bounds.data(), j, per_tile, samples_per_row, m), below);
    };
    *apart = *longest = 0;
    for (int64_t r = 0; r < runs; ++r)
        for (int64_t j = 0; j < tiles; ++j) {
            const int64_t x = begin(r, j), y = begin(r, j + 1);
            if (y < x || y > bounds[r + 1])
                return -1;
            *longest = std::max(*longest, y - x);
            if (r > 0 && y > x && x > bounds[r]) // how far the tile's first id is from that of run 0's tile
                *apart = std::max(*apart, std::abs((int64_t)ids[x] - ids[std::min(begin(0, j), bounds[1] - 1)]));
        }
    return runs;
}

extern "C" int64_t probe(int s, int64_t m) { return probe_place(s, m); }
extern "C" int64_t sample(int s, int64_t m) { return sample_place(s, m); }
