// Feature fetching, the part one GPU does (Sec. 6.2 of arxiv 2311.02909): H_i = the rows of the
// feature matrix H of the vertices in the last frontier, and the forward aggregation of a hop.
//
// Both move rows of f floats, 16 bytes per lane and access whatever f is (rows need only be aligned to 4 bytes; the last
// access of a row ends with the row and may overlap the one before it).  The accesses of a tile of rows are numbered
// through and dealt to the lanes in that order, so no lane is idle because f is no power of two.
#include "bms_device.h"
#include "bms_internal.h"

#include <algorithm>

namespace bms {

constexpr int kFeatThreads = 256;
constexpr int kFeatRows = 64;    // rows per tile
constexpr int kFetchUnroll = 4;  // accesses in flight per lane
constexpr int kFetchSamples = 1024;
constexpr int kFetchMostRuns = 512;
constexpr int kFetchBlock = 16;  // consecutive tiles on one die
constexpr int kFetchRows = 128;  // rows per tile of the fetch
static_assert(kFetchRows <= kFeatThreads && kFeatRows < kFeatThreads, "one thread per row of a tile loads its id or extent");

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
// nothing descends, too much does, or the runs differ too much in length.  A minibatch that lies between two samples is
// missed and ids that do not ascend give runs without a meaning: both only cost speed.
__device__ inline int find_runs(const int32_t *__restrict__ ids, int64_t m, int64_t *bounds, int32_t *samples, int32_t *wsum)
{
    constexpr int PER = kFetchSamples / kFeatThreads;
    __shared__ int32_t longest_s;
    const int tid = threadIdx.x;
    auto place = [&](int s) { return (int64_t)s * (m - 1) / (kFetchSamples - 1); };
#pragma unroll
    for (int q = 0; q < PER; ++q)
        samples[q * kFeatThreads + tid] = ids[place(q * kFeatThreads + tid)];
    if (tid == 0)
        longest_s = 0;
    __syncthreads();
    int32_t descents = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int s = tid * PER + q;
        descents += s + 1 < kFetchSamples && samples[s + 1] < samples[s] ? 1 : 0;
    }
    int32_t total;
    int32_t at = block_exclusive_scan<int32_t, kFeatThreads>(descents, wsum, total);
    const int runs = total + 1;
    if (total == 0 || runs > kFetchMostRuns)
        return 1; // the same in every thread
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int s = tid * PER + q;
        if (s + 1 < kFetchSamples && samples[s + 1] < samples[s]) {
            int64_t lo = place(s), hi = place(s + 1); // the first id below samples[s] in (lo, hi]
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
        atomicMax(&longest_s, (int32_t)((bounds[r + 1] - bounds[r]) / kFeatRows));
    __syncthreads();
    return (int64_t)longest_s * kFeatRows <= 4 * (m / runs) ? runs : 1;
}

// First row of tile j of run r, by one wave: the first row of the run whose id is not below that of run 0's row at the same
// share j / tiles of its length.  It lies near the same share of this run, so 64 ids around there are looked at, then the
// 64 after the last one below; only when it does not, the whole run is searched.  A function of (r, j) alone, run's begin
// and end for the first tile and the one past the last: whatever the ids, the tiles of a run cover it.
__device__ inline int64_t tile_begin(const int32_t *__restrict__ ids, const int64_t *bounds, int64_t r, int64_t j, int64_t tiles)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t b = bounds[r], e = bounds[r + 1];
    if (j == 0 || j == tiles)
        return j ? e : b;
    const int64_t guess = b + (e - b) * j / tiles;
    if (r == 0)
        return guess;
    const int32_t v = ids[bounds[0] + (bounds[1] - bounds[0]) * j / tiles];
    const int64_t w = max<int64_t>(guess - kWave * kWave / 2, b);
    const int64_t p = w + lane * kWave;
    const int below = __popcll(__ballot(p < e && ids[min<int64_t>(p, e - 1)] < v));
    int64_t lo = b, hi = e; // the answer is in [lo, hi]
    if (below == 0) {
        if (w == b)
            return b;
        hi = w;
    } else if (below == kWave) {
        lo = w + (kWave - 1) * kWave + 1;
    } else {
        const int64_t q = w + (below - 1) * kWave + 1;
        return min<int64_t>(q + __popcll(__ballot(q + lane < e && ids[min<int64_t>(q + lane, e - 1)] < v)), e);
    }
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (ids[mid] < v)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// out[j, :] = H[ids[j], :].  An id outside [0, n) gives a row of zeros and raises *flag.
// What bounds it is the traffic to memory.  Written once, but read once per minibatch that needs the row -- unless the
// minibatches get to a row at about the same time.  So the stack's runs (minibatches) are cut into equally many tiles at the
// same ids, and tile j of all runs is fetched before tile j + 1 of any, on one die (workgroups go to the 8 dies in turn):
// the tile's rows of H pass through that die's L2 once.  What is written does not stay there (nontemporal stores).
// 32 minibatches of 295 k rows of 100 floats out of 2.4 M (3.8 GB written): 1647 us and 4.8 GB read in the order of the
// stack (1370 with nontemporal stores), 1255 us and 1.3 GB read so.  More work in flight per wave or compute unit gains nothing.
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
    __shared__ int32_t id_l[kFetchRows];
    __shared__ int64_t tile_s[2];
    const int tid = threadIdx.x;
    const uint32_t per_row = (uint32_t)((f + VEC - 1) / VEC);
    const int64_t runs = LARGE ? find_runs(ids, m, bounds, samples, wsum) : 1;
    if (runs == 1) {
        __syncthreads();
        if (tid == 0) {
            bounds[0] = 0;
            bounds[1] = m;
        }
        __syncthreads();
    }
    const int64_t tiles = max<int64_t>((m / runs + kFetchRows - 1) / kFetchRows, 1); // per run
    const int64_t block = min<int64_t>(max<int64_t>(tiles / 64, 1), kFetchBlock);  // consecutive tiles on one die
    const int64_t rounds = (tiles + 8 * block - 1) / (8 * block) * block * runs;   // units per die
    for (int64_t u = blockIdx.x >> 3; u < rounds; u += gridDim.x >> 3) {
        const int64_t r = u % runs, t = u / runs;
        const int64_t j = (t / block * 8 + (blockIdx.x & 7)) * block + t % block;
        if (j >= tiles)
            continue;
        __syncthreads();
        if (tid < 2 * kWave) {
            const int64_t x = tile_begin(ids, bounds, r, j + tid / kWave, tiles);
            if (tid % kWave == 0)
                tile_s[tid / kWave] = x;
        }
        __syncthreads();
        const int64_t j1 = tile_s[1];
        for (int64_t j0 = tile_s[0]; j0 < j1; j0 += kFetchRows) {
            const int nr = (int)min<int64_t>(kFetchRows, j1 - j0);
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
    const int grid = (grid_for(L, (m + kFetchRows - 1) / kFetchRows, 8) + 7) / 8 * 8;
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
// held to 8 waves per SIMD.  2.8 M rows of 5 entries, 100 floats: 1563 -> 1150 us (8.3 GB between L2 and memory, 7.2 TB/s).
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
            const int64_t b = rowptr_l[walk.row], end = rowptr_l[walk.row + 1];
            const uint32_t at = first_float<VEC>(walk.part, f);
            const float *__restrict__ X = a.X + first_l[walk.row] * f + at;
            Vec acc = 0.0f;
            for (int64_t e = b; e < end; e += kAggUnroll) {
                Vec v[kAggUnroll];
#pragma unroll
                for (int u = 0; u < kAggUnroll; ++u)
                    if (e + u < end) {
                        const int32_t c = staged ? col_l[e + u] : a.col[e0 + e + u];
                        v[u] = *reinterpret_cast<const InMemory *>(X + (int64_t)c * f);
                    }
#pragma unroll
                for (int u = 0; u < kAggUnroll; ++u)
                    if (e + u < end) // entry order
                        acc += v[u];
            }
            if (a.mean && end > b)
                acc /= (float)(end - b);
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
    const int grid = grid_for(L, (a.rows + tile_rows - 1) / tile_rows, 8);
    if (a.f >= 4)
        hipLaunchKernelGGL(aggregate_kernel<4>, dim3(grid), dim3(kFeatThreads), 0, L.stream, a, tile_rows);
    else
        hipLaunchKernelGGL(aggregate_kernel<1>, dim3(grid), dim3(kFeatThreads), 0, L.stream, a, tile_rows);
}

} // namespace bms
