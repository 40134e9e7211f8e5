// Feature fetching, the part one GPU does (Sec. 6.2 of arxiv 2311.02909): H_i = the rows of the
// feature matrix H of the vertices in the last frontier, and the forward aggregation of a hop.
//
// Both move rows of f floats, 16 bytes per lane and access whatever f is (rows need only be aligned to 4 bytes; the last
// access of a row ends with the row and may overlap the one before it).  The accesses of a tile of rows are numbered
// through and dealt to the lanes in that order, so no lane is idle because f is no power of two.
#include "bms_device.h"
#include "bms_internal.h"
#include "feature_runs.h"

#include <algorithm>

namespace bms {

constexpr int kFeatThreads = 256;
constexpr int kFeatRows = 64;    // rows per tile
constexpr int kFetchUnroll = 4;  // accesses in flight per lane
constexpr int kFetchBlock = 16;  // consecutive tiles on one die
static_assert(kFetchLanes == kWave && kFetchSamples % kFeatThreads == 0 && kFetchProbes == kFeatThreads, "feature_runs.h");
static_assert(kFetchTile <= kFeatThreads && kFeatRows < kFeatThreads, "one thread per row of a tile loads its id or extent");

// 16 bytes (or 4) of a row in memory
template <int VEC>
using Floats __attribute__((aligned(4))) = float __attribute__((ext_vector_type(VEC)));

// The accesses of a tile's rows in order, kFeatThreads apart: row and first float of access tid, tid + kFeatThreads, ...
struct RowWalk {
    uint32_t row, part, per_row, row_step, part_step;
    __device__ RowWalk(uint32_t per_row_, uint32_t tid) : per_row(per_row_)
    {
        row = tid / per_row;
        part = tid - row * per_row;
        row_step = kFeatThreads / per_row;
        part_step = kFeatThreads - row_step * per_row;
    }
    __device__ void next()
    {
        row += row_step;
        part += part_step;
        if (part >= per_row) {
            part -= per_row;
            ++row;
        }
    }
};
// first float of the row's access number `part`
template <int VEC>
__device__ inline uint32_t first_float(uint32_t part, int32_t f)
{
    return min(part * VEC, (uint32_t)(f - VEC));
}

// Where the minibatches begin in the stacked ids.  The ids of a minibatch ascend, so its first one is smaller than the one
// before it: kFetchSamples ids at equal distances show between which of them that happens, a binary search where.  Every
// workgroup finds the same.  bounds: kFetchMostRuns + 1 places.  Returns the number of runs; 1 (no structure to use) when
// nothing descends, too much does, the ids between two ascending samples are not in order (feature_runs.h), or the runs differ
// too much in length.
__device__ inline int find_runs(const int32_t *__restrict__ ids, int64_t m, int64_t *bounds, int32_t *samples, int32_t *wsum)
{
    constexpr int PER = kFetchSamples / kFeatThreads;
    __shared__ int32_t longest_s, off_s;
    const int tid = threadIdx.x;
    const int probed = probed_sample(tid);
    const int32_t probe = ids[probe_place(probed, m)];
#pragma unroll
    for (int q = 0; q < PER; ++q)
        samples[q * kFeatThreads + tid] = ids[sample_place(q * kFeatThreads + tid, m)];
    if (tid == 0)
        longest_s = off_s = 0;
    __syncthreads();
    int32_t descents = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int s = tid * PER + q;
        descents += s + 1 < kFetchSamples && samples[s + 1] < samples[s] ? 1 : 0;
    }
    const bool ascends = samples[probed] <= samples[probed + 1];
    const bool off = ascends && probe_off(samples[probed], probe, samples[probed + 1]);
    const int counts = __popcll(__ballot(ascends)) << 16 | __popcll(__ballot(off));
    if ((tid & (kWave - 1)) == 0)
        atomicAdd(&off_s, counts);
    int32_t total;
    int32_t at = block_exclusive_scan<int32_t, kFeatThreads>(descents, wsum, total); // (waits for the additions, too)
    const int runs = total + 1;
    if (!runs_likely(total, off_s >> 16, off_s & 0xFFFF))
        return 1; // the same in every thread
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int s = tid * PER + q;
        if (s + 1 < kFetchSamples && samples[s + 1] < samples[s]) {
            int64_t lo = sample_place(s, m), hi = sample_place(s + 1, m); // the first id below samples[s] in (lo, hi]
            while (hi - lo > 1) {
                const int64_t mid = (lo + hi) >> 1;
                if (ids[mid] < samples[s])
                    hi = mid;
                else
                    lo = mid;
            }
            bounds[++at] = hi;
        }
    }
    if (tid == 0) {
        bounds[0] = 0;
        bounds[runs] = m;
    }
    __syncthreads();
    for (int r = tid; r < runs; r += kFeatThreads) // (in tiles: fits 32 bits)
        atomicMax(&longest_s, (int32_t)((bounds[r + 1] - bounds[r]) / kFetchTile));
    __syncthreads();
    return runs_balanced((int64_t)longest_s * kFetchTile, runs, m) ? runs : 1;
}

// out[j, :] = H[ids[j], :].  An id outside [0, n) gives a row of zeros and raises *flag.
// What bounds it is the traffic to memory.  Written once, but read once per minibatch that needs the row -- unless the
// minibatches get to a row at about the same time.  So the stack's runs (minibatches) are cut into equally many tiles at the
// same ids, and tile j of all runs is fetched before tile j + 1 of any, on one die (workgroups go to the 8 dies in turn):
// the tile's rows of H pass through that die's L2 once.  What is written does not stay there (nontemporal stores).
// 32 minibatches of 295 k rows of 100 floats out of 2.4 M (3.8 GB written): 1647 us and 4.8 GB read in the order of the
// stack (1370 with nontemporal stores), 1255 us and 1.3 GB read so.  More work in flight per wave or compute unit gains nothing.
// Ids without an order take the order of the stack: 10 million of 2.4 million ids, 100 floats, 1.53 ms whatever the draw (while
// descents alone decided, every fourth draw took 14.6 ms).
template <int VEC, bool LARGE>
__global__ __launch_bounds__(kFeatThreads, 8) void feature_fetch_kernel(const float *__restrict__ H, int64_t n, int32_t f,
                                                                     const int32_t *__restrict__ ids, int64_t m,
                                                                     float *__restrict__ out, int32_t *flag)
{
    using Vec = float __attribute__((ext_vector_type(VEC)));
    using InMemory = Floats<VEC>;
    __shared__ int32_t samples[kFetchSamples];
    __shared__ int64_t bounds[kFetchMostRuns + 1];
    __shared__ int32_t wsum[kFeatThreads / kWave];
    __shared__ int32_t id_l[kFetchTile];
    __shared__ int64_t tile_s[kFeatThreads / kWave];
    __shared__ double scale[2]; // 1 / tiles per run, samples per row
    const int tid = threadIdx.x;
    const uint32_t per_row = (uint32_t)((f + VEC - 1) / VEC);
    // (in 32 bits: a GPU's memory holds fewer than 2^37 floats, so there are fewer than 2^32 tiles)
    const uint32_t runs = LARGE ? (uint32_t)find_runs(ids, m, bounds, samples, wsum) : 1u;
    const uint32_t tiles = (uint32_t)tiles_per_run(runs, m);
    if (LARGE && tid == 0) {
        scale[0] = 1.0 / (double)tiles;
        scale[1] = (double)(kFetchSamples - 1) / (double)(m - 1);
    }
    const uint32_t block = min(max(tiles / 64, 1u), (uint32_t)kFetchBlock);        // consecutive tiles on one die
    const uint32_t rounds = (tiles + 8 * block - 1) / (8 * block) * block * runs; // units per die
    const uint32_t stride = gridDim.x >> 3, wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid / kWave);
    for (uint32_t u0 = blockIdx.x >> 3; u0 < rounds; u0 += 2 * stride) {
        // two units at a time, a wave for each begin and end
        const uint32_t u = u0 + wave / 2 * stride;
        const uint32_t t = u / runs, r = u - t * runs;
        const uint32_t j = (t / block * 8 + (blockIdx.x & 7)) * block + t % block;
        int64_t x = 0;
        __syncthreads();
        if (u < rounds && j < tiles) {
            const uint32_t at = j + (wave & 1);
            if (!LARGE || runs == 1)
                x = min<int64_t>((int64_t)at * kFetchTile, m);
            else if (at == 0 || at == tiles)
                x = bounds[at ? r + 1 : r];
            else
                x = tile_begin(bounds, r, at, scale[0], tile_value(ids, samples, bounds, at, scale[0], scale[1], m),
                               [&](int64_t p, int64_t step, int64_t e, int64_t v) {
                                   p += (tid & (kWave - 1)) * step;
                                   return (uint64_t)__ballot(p < e && ids[min<int64_t>(p, e - 1)] < v);
                               });
        }
        if (tid % kWave == 0)
            tile_s[wave] = x;
        __syncthreads();
        for (int unit = 0; unit < 4; unit += 2) {
            for (int64_t j0 = tile_s[unit], j1 = tile_s[unit + 1]; j0 < j1; j0 += kFetchTile) {
                const int nr = (int)min<int64_t>(kFetchTile, j1 - j0);
                __syncthreads();
                if (tid < nr) {
                    int32_t id = ids[j0 + tid];
                    if (id < 0 || (int64_t)id >= n) {
                        *flag = 1;
                        id = -1;
                    }
                    id_l[tid] = id;
                }
                __syncthreads();
                const uint32_t accesses = (uint32_t)nr * per_row;
                float *__restrict__ to = out + j0 * f;
                RowWalk walk(per_row, tid);
                for (uint32_t x = tid; x < accesses; x += kFetchUnroll * kFeatThreads) {
                    Vec v[kFetchUnroll];
                    uint32_t dst[kFetchUnroll];
#pragma unroll
                    for (int q = 0; q < kFetchUnroll; ++q) {
                        if (x + q * kFeatThreads < accesses) {
                            const int32_t id = id_l[walk.row];
                            const uint32_t at = first_float<VEC>(walk.part, f);
                            v[q] = 0.0f;
                            if (id >= 0)
                                v[q] = *reinterpret_cast<const InMemory *>(H + (int64_t)id * f + at);
                            dst[q] = walk.row * (uint32_t)f + at;
                        }
                        walk.next();
                    }
#pragma unroll
                    for (int q = 0; q < kFetchUnroll; ++q)
                        if (x + q * kFeatThreads < accesses) {
                            if (LARGE)
                                __builtin_nontemporal_store(v[q], reinterpret_cast<InMemory *>(to + dst[q]));
                            else
                                *reinterpret_cast<InMemory *>(to + dst[q]) = v[q];
                        }
                }
            }
        }
    }
}

__global__ void feature_done_kernel(int64_t *arrived, int64_t arrival)
{
    __hip_atomic_store(arrived, arrival, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

void launch_feature_fetch(const Launch &L, const float *H, int64_t n, int32_t f, const int32_t *ids, int64_t m,
                          float *out, int32_t *flag, int64_t *arrived, int64_t arrival)
{
    if (m <= 0)
        return;
    // Finding the runs takes a workgroup about 15 us: worth it from some 100 MB on.  Less than that is left in the caches for
    // whoever reads it next.
    const bool large = m >= 64 * kFetchSamples && m * (int64_t)f * 4 >= (100LL << 20);
    const int grid = (grid_for(L, (m + kFetchTile - 1) / kFetchTile, 8) + 7) / 8 * 8;
    void (*const kernels[2][2])(const float *, int64_t, int32_t, const int32_t *, int64_t, float *, int32_t *) = {
        {feature_fetch_kernel<1, false>, feature_fetch_kernel<1, true>}, {feature_fetch_kernel<4, false>, feature_fetch_kernel<4, true>}};
    hipLaunchKernelGGL(kernels[f >= 4][large], dim3(grid), dim3(kFeatThreads), 0, L.stream, H, n, f, ids, m, out, flag);
    hipLaunchKernelGGL(feature_done_kernel, dim3(1), dim3(1), 0, L.stream, arrived, arrival);
}

// Forward neighbourhood aggregation of one hop (Sec. 6.2): the SpMM between the stacked sampled adjacency
// (all entries 1) and the feature rows of its columns.  The row's entries are added in ascending order in fp32.
// mean != 0 divides by the number of entries (rows without entries give zeros).
// Bound by the traffic of the gathered rows (an entry moves whole 128-byte lines).  A tile's row extents and columns go to LDS
// first, so that the gathered rows are one trip to memory away; up to 8 entries of a row are in flight, and registers are
// held to 8 waves per SIMD (places in the tile in 32 bits: in 64 two registers spill).  2.8 M rows of 5 entries, 100 floats: 1563
// -> 1150 us (8.3 GB between L2 and memory, 7.2 TB/s).
constexpr int kAggUnroll = 8;
constexpr int kAggCols = 2048; // columns of a tile in LDS; longer tiles read them from memory
template <int VEC>
__global__ __launch_bounds__(kFeatThreads, 8) void aggregate_kernel(AggArgs a, int tile_rows)
{
    using Vec = float __attribute__((ext_vector_type(VEC)));
    using InMemory = Floats<VEC>;
    __shared__ int64_t rowptr_l[kFeatRows + 1];
    __shared__ int64_t first_l[kFeatRows]; // first column of the row's minibatch
    __shared__ int32_t col_l[kAggCols];
    const int tid = threadIdx.x;
    const int32_t f = a.f;
    const uint32_t per_row = (uint32_t)((f + VEC - 1) / VEC);
    for (int64_t r0 = (int64_t)blockIdx.x * tile_rows; r0 < a.rows; r0 += (int64_t)gridDim.x * tile_rows) {
        const int nr = (int)min<int64_t>(tile_rows, a.rows - r0);
        const int64_t e0 = a.rowptr[r0], entries = a.rowptr[r0 + nr] - e0;
        const bool staged = entries <= kAggCols;
        __syncthreads();
        if (tid <= nr)
            rowptr_l[tid] = a.rowptr[r0 + tid] - e0;
        if (tid < nr)
            first_l[tid] = a.mb_coloff[locate_segment(a.mb_rowoff, a.k, r0 + tid)];
        if (staged)
            for (int e = tid; e < (int)entries; e += kFeatThreads)
                col_l[e] = a.col[e0 + e];
        __syncthreads();
        const uint32_t accesses = (uint32_t)nr * per_row;
        RowWalk walk(per_row, tid);
        for (uint32_t x = tid; x < accesses; x += kFeatThreads, walk.next()) {
            const int64_t b = rowptr_l[walk.row];
            const uint32_t length = (uint32_t)(rowptr_l[walk.row + 1] - b); // (fewer than n)
            const uint32_t at = first_float<VEC>(walk.part, f);
            const float *__restrict__ X = a.X + first_l[walk.row] * f + at;
            Vec acc = 0.0f;
            for (uint32_t e = 0; e < length; e += kAggUnroll) {
                Vec v[kAggUnroll];
#pragma unroll
                for (int u = 0; u < kAggUnroll; ++u)
                    if (e + u < length) {
                        const int32_t c = staged ? col_l[(uint32_t)b + e + u] : a.col[e0 + b + e + u];
                        v[u] = *reinterpret_cast<const InMemory *>(X + (int64_t)c * f);
                    }
#pragma unroll
                for (int u = 0; u < kAggUnroll; ++u)
                    if (e + u < length) // entry order
                        acc += v[u];
            }
            if (a.mean && length)
                acc /= (float)length;
            *reinterpret_cast<InMemory *>(a.out + (r0 + walk.row) * f + at) = acc;
        }
    }
}

void launch_aggregate(const Launch &L, const AggArgs &a)
{
    if (a.rows <= 0)
        return;
    int tile_rows = kFeatRows; // fewer where that leaves workgroups without a tile or with one more than others
    while (tile_rows > 4 && a.rows < (int64_t)tile_rows * L.num_cu * 64 && tile_rows * ((a.f + 3) / 4) > kFeatThreads)
        tile_rows /= 2;
    // A tile per workgroup, except where a tile's accesses keep all threads busy to its end: then eight workgroups per compute unit that go
    // on are level or faster, as the next tile costs less than the next workgroup.  Going on and a tile each, hops of 0.4 and 1.5 M rows of 5
    // entries: 5 floats 32.3 and 31.0 us, 104.5 and 97.2; 20 53.5 and 52.5, 194 and 187; 100 160 and 156, 590 and 575; 32 47.6 and 51.7, 184
    // and 188; 64 97 and 104, 335 and 339; 128 173 and 177, 656 and 655.
    const bool full = tile_rows * (a.f >= 4 ? (a.f + 3) / 4 : a.f) % kFeatThreads == 0;
    const int grid = grid_for(L, (a.rows + tile_rows - 1) / tile_rows, full ? 8 : kOnePass);
    if (a.f >= 4)
        hipLaunchKernelGGL(aggregate_kernel<4>, dim3(grid), dim3(kFeatThreads), 0, L.stream, a, tile_rows);
    else
        hipLaunchKernelGGL(aggregate_kernel<1>, dim3(grid), dim3(kFeatThreads), 0, L.stream, a, tile_rows);
}

} // namespace bms
