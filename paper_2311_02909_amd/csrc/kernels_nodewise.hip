// Node-wise (GraphSAGE) bulk sampling kernels, Sec. 4.1 of arxiv 2311.02909.
//
// One hop over the stacked frontier (all k minibatches at once, Eq. 1):
//   nw_rows    P = Q A: Q has one nonzero per row, so row r of P is the CSR row of the frontier
//              vertex; only its extent (begin, degree) is fetched.  Also the per-tile sums of
//              min(degree, s) that size the output rows.
//   (scan)     exclusive scan of the tile sums -> where each tile's output starts
//   nw_sample  SAMPLE: per row, min(degree, s) distinct positions (ITS without replacement,
//              Sec. 4.1.2), the chosen neighbours gathered, staged through LDS and written
//              coalesced as global ids
// EXTRACT (Sec. 4.1.3: distinct sampled ids ascending = next frontier, global id -> local column) is
// done by the kernels of kernels_dedup_sort.hip / kernels_dedup.hip.  The first design of it lives
// here and serves vertex ranges too wide for those: nw_sample also sets the ids' bits in a
// per-minibatch vertex set in HBM, the set is ranked (kernels_common.hip), and
//   nw_relabel global id -> local column index = rank in the minibatch's vertex set
// Variant (the frontier's own vertices stay columns): every row carries its own vertex as one more
// entry through EXTRACT, and nw_strip_self takes it out of the row again afterwards.
// Variant (independent draws): the s draws of a row are each an integer in [0, degree), the row keeps
// the distinct picks; its length is only known after the draws, so nw_rows makes them too.
#include "bms_device.h"
#include "bms_internal.h"
#include "nw_draws.h"

#include <algorithm>

namespace bms {

// Independent draws (replace_draws) for any s <= kMaxSampledFanout by one wave: the draws are written to `buf` (LDS, room for the next
// power of two >= max(s, 64)), sorted there by a bitonic network, and the distinct values moved down to
// buf[0..m) in ascending order.  Returns m (the same value in every lane).
__device__ inline int32_t wave_replace_draws(volatile uint32_t *buf, uint64_t key, uint32_t deg, int32_t s, int lane)
{
    int32_t P = kWave;
    while (P < s)
        P <<= 1;
    for (int32_t j = lane; j < P; j += kWave)
        buf[j] = j < s ? bounded32(draw32(key, (uint32_t)j), deg) : 0xFFFFFFFFu; // padding sorts last (deg < 2^31)
    __builtin_amdgcn_wave_barrier();
    for (int32_t size = 2; size <= P; size <<= 1) {
        for (int32_t stride = size >> 1; stride > 0; stride >>= 1) {
            for (int32_t t = lane; t < P / 2; t += kWave) {
                const int32_t lo = ((t & ~(stride - 1)) << 1) | (t & (stride - 1)); // bit `stride` clear
                const int32_t hi = lo | stride;
                const bool up = (lo & size) == 0;
                const uint32_t x = buf[lo], y = buf[hi];
                if ((x > y) == up) {
                    buf[lo] = y;
                    buf[hi] = x;
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    int32_t m = 0;
    uint32_t last = 0; // value before this chunk's first one
    for (int32_t base = 0; base < P; base += kWave) {
        const int32_t j = base + lane;
        const uint32_t v = buf[j];
        uint32_t prev = __shfl_up(v, 1);
        if (lane == 0)
            prev = last;
        const bool head = j < s && (j == 0 || v != prev);
        const uint64_t heads = __ballot(head);
        __builtin_amdgcn_wave_barrier(); // the chunk is read before any of it is overwritten (targets are <= sources)
        if (head)
            buf[m + __popcll(heads & ((1ull << lane) - 1ull))] = v;
        m += __popcll(heads);
        last = __shfl(v, kWave - 1);
        __builtin_amdgcn_wave_barrier();
    }
    return m;
}

// The row tiles that a wave or workgroup visits: of all minibatches, in order of their place in the minibatch, minibatch by
// minibatch within a step.
//   stacked: tile j of every minibatch in step j, the steps dealt out to all of the launch's workgroups in turn
//   by dies: `most` steps, the number that the largest minibatch has, those of a smaller one spread evenly, and each die takes an
//            eighth of that order.  The rows of a minibatch ascend by vertex id, so what runs at the same time on a die touches
//            one part of the id range in all minibatches: a line that several minibatches need is fetched once and is in the
//            die's own cache when the next one asks.
// Each has kernels of its own: by dies a workgroup computes for half a microsecond before its first read (one minibatch, 74 seeds,
// (13, 19): a call 72.9 us with both in one kernel, 72.2 so; the second hop's sampling of 7 x 653, (13, 11): 8.4 to 9.0 and 8.0).
constexpr int kDies = 8;
template <bool DIES>
struct TileWalk {
    int32_t k, i, step_i, left; // i: minibatch; left: visits, by dies
    int64_t j, most, step_j;
    // workgroups are dealt to the dies in turn; wave `part` of `parts` in the workgroup; by dies gridDim.x is a multiple of kDies
    __device__ TileWalk(const NwHop &a, uint32_t part, uint32_t parts) : k(a.k), left(0), most(uniform_load(a.mb_tileoff + a.k + 1))
    {
        const uint32_t step = (DIES ? gridDim.x / kDies : gridDim.x) * parts;
        step_j = scalar(step / (uint32_t)k);
        step_i = (int32_t)(step - (uint32_t)step_j * (uint32_t)k);
        if (!DIES) {
            const uint32_t pos = blockIdx.x * parts + part, q = scalar(pos / (uint32_t)k);
            j = q;
            i = (int32_t)(pos - q * (uint32_t)k);
            return;
        }
        const int64_t items = most * k, per = (items + kDies - 1) / kDies;
        const int64_t lo = (blockIdx.x % kDies) * per, hi = min<int64_t>(lo + per, items);
        const int64_t pos = lo + (blockIdx.x / kDies) * parts + part;
        if (pos < hi && hi >> 31 == 0) { // (divisions of 64 bits are half a microsecond at the start of a workgroup)
            left = (int32_t)((uint32_t)(hi - pos + step - 1) / step);
            j = (uint32_t)pos / (uint32_t)k;
            i = (int32_t)((uint32_t)pos - (uint32_t)j * (uint32_t)k);
        } else {
            if (pos < hi)
                left = (int32_t)((hi - pos + step - 1) / step);
            i = (int32_t)(pos % k);
            j = pos / k;
        }
    }
    __device__ bool more() const { return DIES ? left > 0 : j < most; }
    __device__ void next()
    {
        --left;
        i += step_i;
        j += step_j;
        if (i >= k) {
            i -= k;
            ++j;
        }
    }
    // number of the tile among all, or -1 when the minibatch has none at this step; its rows
    __device__ int64_t tile(const NwHop &a, int64_t &r0, int32_t &rows) const
    {
        int64_t t0 = uniform_load(a.mb_tileoff + i), t1 = uniform_load(a.mb_tileoff + i + 1);
        const int64_t row0 = uniform_load(a.mb_rowoff + i), row1 = uniform_load(a.mb_rowoff + i + 1);
        asm volatile("" : "+s"(t0), "+s"(t1) : "s"(row0), "s"(row1)); // (all on their way at once, the rows not a trip to memory later)
        const int64_t tiles = t1 - t0;
        const bool apart = DIES && most < 65536 && tiles != most; // (of larger minibatches: tile q in step q)
        int64_t jj = j;
        if (apart) // tile q is visited in step floor(q most / tiles)
            jj = ((uint32_t)j * (uint32_t)tiles + (uint32_t)most - 1u) / (uint32_t)most;
        if (jj >= tiles || (apart && ((uint32_t)jj * (uint32_t)most) / (uint32_t)tiles != j))
            return -1;
        r0 = row0 + jj * kRowTile;
        rows = row1 - r0 < kRowTile ? (int32_t)(row1 - r0) : kRowTile;
        return t0 + jj;
    }
};

// S = 0: rows keep min(degree, s) entries.  S > 0: independent draws, s <= S; the row's length is the number
// of distinct picks.
// What bounds it is the number of rowptr lines on their way.  A wave takes a tile of its own, four rows per lane, and needs no
// barrier.  Two hops each: 256 x 1024 seeds, (15, 10, 5), 111 M vertices: 265 -> 235 us; 128 minibatches on 8.7 M vertices:
// 236 -> 186 us; 64 on 2.4 M: 71 -> 56 us.  Of workgroups per compute unit that go from tile to tile, 4 are best: 1, 2, 4 and 16 take
// 238, 199, 186 and 193 us (8.7 M vertices), 77, 63, 56 us (2.4 M): fewer have too few lines on their way, more drift apart over a
// larger part of the ids.  Started in order with a tile per wave they stay together: 180 -> 174 us, 57 -> 55, 220 either way (111 M).
constexpr int kTileRounds = kRowTile / kWave;
template <int S>
__global__ __launch_bounds__(kRowTile) void nw_rows_kernel(NwHop a)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    for (int64_t q = (int64_t)blockIdx.x * kRowTile + tid; q < a.zero_quads; q += (int64_t)gridDim.x * kRowTile)
        a.zero[q] = make_uint4(0, 0, 0, 0);
    for (TileWalk<true> walk(a, scalar((uint32_t)(tid / kWave)), kRowTile / kWave); walk.more(); walk.next()) {
        int64_t r0;
        int32_t rows;
        const int64_t t = walk.tile(a, r0, rows);
        if (t < 0)
            continue;
        const int32_t *__restrict__ from = a.row_vertex + r0;
        int32_t v[kTileRounds];
#pragma unroll
        for (int u = 0; u < kTileRounds; ++u)
            v[u] = u * kWave + lane < rows ? from[u * kWave + lane] : -1;
        int64x2_a8 extent[kTileRounds];
#pragma unroll
        for (int u = 0; u < kTileRounds; ++u) {
            extent[u] = int64x2_a8{0, 0};
            if (v[u] >= 0 && (int64_t)v[u] < a.n) // seeds are verified separately; never read out of bounds
                extent[u] = row_extent(a.A_rowptr, v[u]);
        }
        int64_t cnt = 0;
#pragma unroll
        for (int u = 0; u < kTileRounds; ++u) {
            if (u * kWave + lane >= rows)
                continue;
            const int32_t deg = (int32_t)(extent[u][1] - extent[u][0]);
            a.row_beg[r0 + u * kWave + lane] = extent[u][0];
            a.row_deg[r0 + u * kWave + lane] = deg;
            if (S == 0) {
                cnt += deg < a.s ? deg : a.s;
            } else if (deg > 0) {
                uint32_t c[S > 0 ? S : 1];
                cnt += replace_draws(row_key(a.hopkey, a.mb_base + (uint32_t)walk.i, (uint32_t)v[u]), (uint32_t)deg, a.s, c);
            }
            cnt += a.self_entry;
        }
        const uint32_t low = wave_inclusive_scan_dpp((uint32_t)cnt & 0xFFFFFFu), high = wave_inclusive_scan_dpp((uint32_t)(cnt >> 24));
        if (lane == kWave - 1)
            a.tile_off[t] = ((int64_t)high << 24) + low;
    }
}

// Independent draws with s > 32: extents by one row per lane as above, then one row per wave: draws sorted (across the
// lanes for s <= 64, in LDS above), distinct ones counted; the count is kept per row (row_cnt) so that the sampling
// kernel can place the rows before it repeats the draws.
constexpr int kWideRowsThreads = 1024;
template <bool LANES>
__global__ __launch_bounds__(kWideRowsThreads) void nw_rows_replace_wide_kernel(NwHop a)
{
    constexpr int NW = kWideRowsThreads / kWave;
    __shared__ uint32_t chosen_all[LANES ? 1 : NW * kMaxSampledFanout];
    __shared__ int64_t wsum[kRowTile / kWave];
    __shared__ int32_t deg_of[kRowTile], vert_of[kRowTile], cnt_of[kRowTile];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    volatile uint32_t *buf = chosen_all + (LANES ? 0 : wave * kMaxSampledFanout);
    for (int64_t q = (int64_t)blockIdx.x * kWideRowsThreads + tid; q < a.zero_quads; q += (int64_t)gridDim.x * kWideRowsThreads)
        a.zero[q] = make_uint4(0, 0, 0, 0);
    const int64_t most = a.mb_tileoff[a.k + 1];
    for (int64_t v = blockIdx.x; v < most * a.k; v += gridDim.x) {
        const int i = (int)(v % a.k);
        const int64_t j = v / a.k;
        if (j >= a.mb_tileoff[i + 1] - a.mb_tileoff[i])
            continue;
        const int64_t t = a.mb_tileoff[i] + j;
        const int64_t r0 = a.mb_rowoff[i] + j * kRowTile;
        const int64_t r = r0 + tid;
        const int64_t left = a.mb_rowoff[i + 1] - r0;
        const int nr = (int)(left < kRowTile ? left : kRowTile);
        if (tid < nr) {
            const int32_t vtx = a.row_vertex[r];
            int64_t beg = 0, deg = 0;
            if (vtx >= 0 && (int64_t)vtx < a.n) {
                beg = a.A_rowptr[vtx];
                deg = a.A_rowptr[vtx + 1] - beg;
            }
            a.row_beg[r] = beg;
            a.row_deg[r] = (int32_t)deg;
            deg_of[tid] = (int32_t)deg;
            vert_of[tid] = vtx;
        }
        __syncthreads();
        for (int q = wave; q < nr; q += NW) {
            int32_t m = 0;
            if (deg_of[q] > 0) {
                const uint64_t key = row_key(a.hopkey, a.mb_base + (uint32_t)i, (uint32_t)vert_of[q]);
                uint32_t pos;
                m = LANES ? wave_replace_draws64(key, (uint32_t)deg_of[q], a.s, lane, pos)
                          : wave_replace_draws(buf, key, (uint32_t)deg_of[q], a.s, lane);
            }
            if (lane == 0)
                cnt_of[q] = m;
        }
        __syncthreads();
        if (tid < kRowTile) {
            int64_t cnt = 0;
            if (tid < nr) {
                a.row_cnt[r] = cnt_of[tid];
                cnt = cnt_of[tid] + a.self_entry;
            }
            cnt = wave_sum(cnt);
            if (lane == 0)
                wsum[wave] = cnt;
        }
        __syncthreads();
        if (tid == 0) {
            int64_t tot = 0;
#pragma unroll
            for (int w = 0; w < kRowTile / kWave; ++w)
                tot += wsum[w];
            a.tile_off[t] = tot;
        }
        __syncthreads();
    }
}

// Visits that a walk by dies is likely to have: k times the tiles of the largest minibatch, taken to be an eighth and three tiles more
// than the mean (of 6 minibatches with 40 tiles, one tile too few for the largest had a wave go on to a second one: 5.0 -> 6.6 us).
// Nothing depends on it: where there are more, workgroups go on to another tile.
static int64_t likely_visits(const NwHop &a)
{
    const int64_t tiles = a.rows_tune / a.k / kRowTile;
    return (int64_t)a.k * (tiles + tiles / 8 + 3);
}

void launch_nw_rows(const Launch &L, const NwHop &a)
{
    const int64_t tiles = std::max(a.rows_bound / kRowTile + a.k, a.zero_quads / (8 * kRowTile));
    // A tile per wave as a rule, of as many as the minibatches had in the call before; of a bound of the rows, four workgroups per
    // compute unit, and also of minibatches with less than a tile on average, most of whose likely visits have none (20000 x 8 seeds,
    // (4, 4): two hops 23.6 us, 28.4 with a wave for each of them).
    const bool one_each = a.rows_tune < a.rows_bound && a.rows_tune >= (int64_t)a.k * kRowTile;
    const int64_t wgs = std::max((one_each ? likely_visits(a) : a.rows_bound / kRowTile + a.k) / (kRowTile / kWave) + 1, a.zero_quads / (8 * kRowTile));
    const dim3 grid((grid_for(L, wgs, one_each ? kOnePass : 4) + kDies - 1) / kDies * kDies), block(kRowTile);
    if (!a.replace)
        hipLaunchKernelGGL(nw_rows_kernel<0>, grid, block, 0, L.stream, a);
    else if (a.s <= 4)
        hipLaunchKernelGGL(nw_rows_kernel<4>, grid, block, 0, L.stream, a);
    else if (a.s <= 8)
        hipLaunchKernelGGL(nw_rows_kernel<8>, grid, block, 0, L.stream, a);
    else if (a.s <= 16)
        hipLaunchKernelGGL(nw_rows_kernel<16>, grid, block, 0, L.stream, a);
    else if (a.s <= 32)
        hipLaunchKernelGGL(nw_rows_kernel<32>, grid, block, 0, L.stream, a);
    else if (a.s <= kWave)
        hipLaunchKernelGGL(nw_rows_replace_wide_kernel<true>, dim3(grid_for(L, tiles, 2)), dim3(kWideRowsThreads), 0, L.stream, a);
    else
        hipLaunchKernelGGL(nw_rows_replace_wide_kernel<false>, dim3(grid_for(L, tiles, 1)), dim3(kWideRowsThreads), 0, L.stream, a);
}

// Sum of the tiles before tile t, for all threads of a workgroup (sum_tiles); `room`: a word per wave.  Up to four sums per thread
// out of L2 instead of a launch of the scan.  Calls of (15, 10, 5) for one minibatch of 1024 seeds 139 -> 134 us, (40, 40) for 8 of
// 512 205 -> 193; with 1950 tiles, twice what the chip has workgroups for, 721 -> 726, so not more than kMostSummedTiles.
__device__ __forceinline__ int64_t tiles_before(const NwHop &a, int64_t t, int64_t *room)
{
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid)); // (places: computed anew for every tile, not kept in registers)
    constexpr int kEach = kMostSummedTiles / kRowTile; // consecutive ones, two to a read (tile t itself may be read)
    const int left = (int)t - (int)tid * kEach;
    const longlong2 *from = reinterpret_cast<const longlong2 *>(a.tile_off) + tid * (kEach / 2);
    longlong2 two[kEach / 2];
#pragma unroll
    for (int u = 0; u < kEach / 2; ++u) {
        two[u] = make_longlong2(0, 0);
        if (2 * u < left)
            two[u] = from[u];
    }
    int64_t sum = 0;
#pragma unroll
    for (int u = 0; u < kEach / 2; ++u)
        sum += two[u].x + (2 * u + 1 < left ? two[u].y : 0);
    // 64 lanes' sums of low and of high bits fit 32 bits each (a tile has fewer than 2^40 entries)
    const uint32_t low = wave_inclusive_scan_dpp((uint32_t)sum & 0xFFFFFFu), high = wave_inclusive_scan_dpp((uint32_t)(sum >> 24));
    __syncthreads();
    if ((tid & (kWave - 1)) == kWave - 1)
        room[tid / kWave] = ((int64_t)high << 24) + low;
    __syncthreads();
    sum = 0;
#pragma unroll
    for (int w = 0; w < kRowTile / kWave; ++w)
        sum += room[w];
    return sum;
}

// entries in all, by one thread of the launch
__device__ __forceinline__ void leave_total(const NwHop &a, int64_t total)
{
    *a.nnz_out = total;
    a.out_rowptr[a.mb_rowoff[a.k]] = total;
}

// ---------------------------------------------------------------------------------------------
// SAMPLE, one row per lane, fanout <= S (compile-time capacity of the per-lane position list; S > 32: launch_nw_sample_impl).
//
// Draws: nw_draws.h.
//
// What bounds it is the number of memory lines that a compute unit can wait for at a time (about 92, by the counters: reads
// times latency over time), so what counts is how few lines are asked for, and how near they are.  The chosen positions are
// laid out in LDS first and read with the picks of a row in neighbouring lanes: picks on one line are one request, where a
// lane that reads its row's picks one after the other asks for the line again unless the compute unit's 32 KB still hold it.
// Last hop of 256 x 1024 seeds, (15, 10, 5), 111 M vertices: 943 us so far, 856 us by the layout, 742 us with four workgroups
// per compute unit as well (launch_nw_sample_impl); 128 minibatches on 8.7 M vertices of 154 times the degree: 1429 -> 1123 us.
// ---------------------------------------------------------------------------------------------
constexpr uint32_t kSelfMark = 0x80000000u; // staged entry: a vertex id, not a place in A_col
// SUM: a.sum_tiles; kernels of their own, as the sums' registers would cost the others a workgroup per compute unit
template <int S, bool SET, bool REPLACE, bool SUM, bool DIES>
__global__ __launch_bounds__(kRowTile) void nw_sample_kernel(NwHop a, VSet vs)
{
    __shared__ uint32_t stage[kRowTile * (S + 1)]; // + 1: the row's own vertex when rows carry it
    __shared__ int32_t wsum[kRowTile / kWave];
    __shared__ int64_t tsum[SUM ? kRowTile / kWave : 1];
    __shared__ uint32_t seg_hist[kMaxFusedSegments]; // sampled ids per id-range segment, of this workgroup's minibatch
    __shared__ uint16_t seg_tab_l[kMaxCells + 1];    // segment of every cell of ids, when the segments differ in width
    const int tid = threadIdx.x;
    const int32_t s = a.s;
    const bool count = a.seg_cnt != nullptr; // by dies after every tile; else gridDim.x is a multiple of k: every tile of this
                                             // workgroup belongs to minibatch blockIdx.x % k
    const bool by_table = count && a.seg_tab != nullptr;
    const bool flat = a.flat != 0;
    const uint32_t self_mark = a.self_entry ? kSelfMark : 0u;
    if (count) {
        for (int c = tid; c < a.seg_C; c += kRowTile)
            seg_hist[c] = 0;
        if (by_table)
            for (int x = tid; x <= kMaxCells; x += kRowTile)
                seg_tab_l[x] = a.seg_tab[x];
        __syncthreads();
    }
    auto leave_counts = [&](int i) { // (barriers between this and the next tile's additions)
        uint32_t *__restrict__ out = a.seg_cnt + (int64_t)i * a.seg_C;
        for (int c = tid; c < a.seg_C; c += kRowTile)
            if (seg_hist[c]) {
                atomicAdd(&out[c], seg_hist[c]);
                seg_hist[c] = 0;
            }
    };
    // the extent of the lane's row in the workgroup's next tile is fetched while the current tile is sampled
    TileWalk<DIES> walk(a, 0, 1);
    int64_t t, t_next, r0, r0_next;
    int32_t rows, rows_next;
    int64_t beg, beg_next;
    int32_t deg, deg_next;
    auto extent = [&](int64_t &t, int64_t &r0, int32_t &rows, int64_t &beg, int32_t &deg) {
        t = -1;
        r0 = beg = 0;
        rows = deg = 0;
        if (walk.more())
            t = walk.tile(a, r0, rows);
        if (t >= 0 && tid < rows) {
            beg = a.row_beg[r0 + tid];
            deg = a.row_deg[r0 + tid];
        }
    };
    if (SUM && walk.most == 0 && blockIdx.x == 0 && tid == 0)
        leave_total(a, 0);
    extent(t, r0, rows, beg, deg);
    for (; walk.more(); t = t_next, r0 = r0_next, rows = rows_next, beg = beg_next, deg = deg_next) {
        const int i = walk.i;
        walk.next();
        extent(t_next, r0_next, rows_next, beg_next, deg_next);
        if (t < 0)
            continue;
        const int64_t r = r0 + tid;
        const bool valid = tid < rows;
        int32_t cnt = 0;
        uint32_t c[S];
        if (valid) {
            if (!REPLACE)
                cnt = deg < s ? deg : s;
            else if (deg > 0) // independent draws: the row's length is the number of distinct picks
                cnt = replace_draws(row_key(a.hopkey, a.mb_base + (uint32_t)i, (uint32_t)a.row_vertex[r]),
                                    (uint32_t)deg, s, c);
        }
        int32_t tot;
        const int32_t loc = block_exclusive_scan<int32_t, kRowTile>(valid ? cnt + a.self_entry : 0, wsum, tot);
        const int64_t base = SUM ? tiles_before(a, t, tsum) : a.tile_off[t];
        if (SUM && tid == 0 && t == a.mb_tileoff[a.k] - 1)
            leave_total(a, base + tot);
        if (valid)
            a.out_rowptr[r] = base + loc;
        if (SET && valid && a.mark_self) {
            const int32_t self = a.row_vertex[r];
            if (self >= 0 && (int64_t)self < a.n)
                atomicOr(&vs.words[(int64_t)i * vs.nw + (self >> 5)], 1u << (self & 31));
        }
        if (valid && a.self_entry) { // a seed outside [0, n) is reported by the seed check; EXTRACT still gets a valid id
            const int32_t self = a.row_vertex[r];
            stage[loc + cnt] = ((self >= 0 && (int64_t)self < a.n) ? (uint32_t)self : 0u) | (flat ? kSelfMark : 0u);
        }
        if (cnt > 0) {
            if (!REPLACE && deg > s)
                distinct_draws<S>(row_key(a.hopkey, a.mb_base + (uint32_t)i, (uint32_t)a.row_vertex[r]), (uint32_t)deg, s, c);
            const int32_t *__restrict__ src = a.A_col + beg;
            int32_t m = 0;
#pragma unroll
            for (int j = 0; j < S; ++j) {
                const uint32_t at = !REPLACE && deg <= s ? (uint32_t)j : c[j];
                if (REPLACE ? (j < s && (j == 0 || c[j] != c[j - 1])) : j < cnt)
                    stage[loc + m++] = flat ? (uint32_t)beg + at : (uint32_t)src[at];
            }
        }
        __syncthreads();
        uint32_t *__restrict__ words = vs.words + (int64_t)i * vs.nw;
        // Whole lines of the output to a store, where neither atomics nor the draws bound it.  Calls without and with it, on 2.4 M
        // vertices: 64 x 1024 seeds, (15, 10, 5) 626 and 612 us, (4, 4, 4) 205 and 206; 32 x 1024, (15, 15, 3) 430 and 424, (16, 16)
        // 163 and 164; on 0.3 M, 32 x 1024, (16, 16) 102.1 and 103.5; on 8.7 M, (15, 10, 5) 852 and 853.  Of more than 16: 32 x 1024,
        // (20, 20) 208 and 214, 64 x 512, (10, 30) 162 and 166, on 0.3 M, 32 x 512, (30, 30) 124 and 127
        constexpr bool LINES = !SET && S <= 16;
        constexpr int kGatherUnroll = LINES ? 6 : 5;
        const int32_t head = LINES ? (int32_t)(base & 31) : 0;
        for (int32_t e0 = tid - head; e0 < tot; e0 += kGatherUnroll * kRowTile) {
            uint32_t g[kGatherUnroll];
#pragma unroll
            for (int u = 0; u < kGatherUnroll; ++u) {
                const int32_t e = e0 + u * kRowTile;
                if (e < tot && (!LINES || e >= 0)) {
                    g[u] = stage[e];
                    if (flat)
                        g[u] = (g[u] & self_mark) ? g[u] & ~kSelfMark : (uint32_t)a.A_col[g[u]];
                }
            }
#pragma unroll
            for (int u = 0; u < kGatherUnroll; ++u) {
                const int32_t e = e0 + u * kRowTile;
                if (e < tot && (!LINES || e >= 0)) {
                    a.out_col[base + e] = (int32_t)g[u];
                    if (SET)
                        atomicOr(&words[g[u] >> 5], 1u << (g[u] & 31u));
                    if (count)
                        atomicAdd(&seg_hist[by_table ? (uint32_t)seg_tab_l[g[u] >> a.seg_shift] : g[u] >> a.seg_shift], 1u);
                }
            }
        }
        __syncthreads();
        if (DIES && count)
            leave_counts(i);
    }
    if (!DIES && count)
        leave_counts((int)(blockIdx.x % a.k));
}

// ---------------------------------------------------------------------------------------------
// SAMPLE, one row per wave, any fanout: rows with degree <= s are copied whole; longer rows keep their sorted chosen
// list across the wave's lanes in K registers (s <= 64 K; nw_draws.h), or, K = 0, in LDS (s <= kMaxSampledFanout).  In
// LDS, for draw j the number c of chosen positions that the pick steps over is the count of list entries p_t with
// p_t - t <= x (p_t - t = unchosen positions before p_t, non-decreasing in t), found by binary search.
// A row's draws are one chain, so what counts is the instructions per draw and how many rows are in progress: across the
// lanes a draw takes about 8 vector instructions and no trip to LDS, and `parts` workgroups share the rows of a tile so
// that hops of few rows still fill the chip.  8 minibatches of 512, fanouts (40, 40), 2.4 M vertices: the two hops took
// 547 + 1353 us with the list in LDS and one workgroup per tile, 9 + 73 us so (the second one row per lane now: launch_nw_sample_impl).
// ---------------------------------------------------------------------------------------------
template <bool SET, bool REPLACE, int K>
__global__ __launch_bounds__(kRowTile) void nw_sample_wide_kernel(NwHop a, VSet vs, int32_t parts)
{
    constexpr int NW = kRowTile / kWave;
    __shared__ uint32_t chosen_all[K ? 1 : NW * kMaxSampledFanout];
    __shared__ int64_t wsum[NW];
    __shared__ int64_t row_loc[kRowTile];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    volatile uint32_t *chosen = chosen_all + (K ? 0 : wave * kMaxSampledFanout);
    const int64_t nwork = a.mb_tileoff[a.k] * parts;
    const int32_t s = a.s;
    if (a.sum_tiles && nwork == 0 && blockIdx.x == 0 && tid == 0)
        leave_total(a, 0);
    for (int64_t v = blockIdx.x; v < nwork; v += gridDim.x) {
        const int64_t t = v / parts;
        const int part = (int)(v % parts);
        const int i = locate_segment(a.mb_tileoff, a.k, t);
        const int64_t r0 = a.mb_rowoff[i] + (t - a.mb_tileoff[i]) * kRowTile;
        const int64_t rend = a.mb_rowoff[i + 1];
        const int64_t r = r0 + tid;
        int64_t cnt = 0;
        if (r < rend) {
            const int64_t deg = a.row_deg[r];
            cnt = (REPLACE ? (int64_t)a.row_cnt[r] : (deg < s ? deg : s)) + a.self_entry;
        }
        int64_t tot;
        const int64_t loc = block_exclusive_scan<int64_t, kRowTile>(cnt, wsum, tot);
        const int64_t base = a.sum_tiles ? tiles_before(a, t, wsum) : a.tile_off[t];
        if (a.sum_tiles && tid == 0 && v == nwork - 1)
            leave_total(a, base + tot);
        if (r < rend && part == 0)
            a.out_rowptr[r] = base + loc;
        row_loc[tid] = base + loc;
        __syncthreads();
        uint32_t *__restrict__ words = vs.words + (int64_t)i * vs.nw;
        for (int q = part * NW + wave; q < kRowTile; q += NW * parts) { // rows of this tile, one per wave
            const int64_t rr = r0 + q;
            if (rr >= rend)
                break;
            const int64_t beg = a.row_beg[rr];
            const int32_t deg = a.row_deg[rr];
            int32_t *__restrict__ dst = a.out_col + row_loc[q];
            const int32_t *__restrict__ src = a.A_col + beg;
            auto put = [&](int32_t e, int32_t g) {
                dst[e] = g;
                if (SET)
                    atomicOr(&words[g >> 5], 1u << (g & 31));
            };
            if (SET && a.mark_self && lane == 0) {
                const int32_t self = a.row_vertex[rr];
                if (self >= 0 && (int64_t)self < a.n)
                    atomicOr(&words[self >> 5], 1u << (self & 31));
            }
            if (a.self_entry && lane == 0) { // the row's own vertex, after its sampled ones (kept inside [0, n):
                                             // a bad seed is reported by the seed check, EXTRACT still gets a valid id)
                int32_t g = a.row_vertex[rr];
                if (g < 0 || (int64_t)g >= a.n)
                    g = 0;
                put(REPLACE ? a.row_cnt[rr] : (deg < s ? deg : s), g);
            }
            if (REPLACE ? deg <= 0 : deg <= s) {
                for (int32_t e = lane; e < deg; e += kWave)
                    put(e, src[e]);
                continue;
            }
            const uint64_t key = row_key(a.hopkey, a.mb_base + (uint32_t)i, (uint32_t)a.row_vertex[rr]);
            if (REPLACE) { // independent draws: the distinct picks, sorted by the wave
                if (K == 1) {
                    uint32_t pos;
                    const int32_t m = wave_replace_draws64(key, (uint32_t)deg, s, lane, pos);
                    if (lane < m)
                        put(lane, src[pos]);
                } else {
                    const int32_t m = wave_replace_draws(chosen, key, (uint32_t)deg, s, lane);
                    for (int32_t e = lane; e < m; e += kWave)
                        put(e, src[chosen[e]]);
                    __builtin_amdgcn_wave_barrier();
                }
                continue;
            }
            if (K > 0) {
                uint32_t pos[K ? K : 1];
                wave_distinct_draws<(K ? K : 1)>(key, (uint32_t)deg, s, lane, pos);
#pragma unroll
                for (int u = 0; u < K; ++u)
                    if (64 * u + lane < s)
                        put(64 * u + lane, src[pos[u]]);
                continue;
            }
            for (int32_t j = 0; j < s; ++j) {
                const uint32_t x = bounded32(draw32(key, (uint32_t)j), (uint32_t)deg - (uint32_t)j);
                // c = number of t in [0,j) with chosen[t] - t <= x   (all lanes compute the same value)
                int32_t lo = 0, hi = j;
                while (lo < hi) {
                    const int32_t mid = (lo + hi) >> 1;
                    if (chosen[mid] - (uint32_t)mid <= x)
                        lo = mid + 1;
                    else
                        hi = mid;
                }
                const int32_t c = lo;
                // shift chosen[c..j) up by one, top chunk first so nothing is overwritten before it is read
                for (int32_t top = j; top > c; top -= kWave) {
                    const int32_t idx = top - 1 - lane; // source index
                    uint32_t val = 0;
                    if (idx >= c)
                        val = chosen[idx];
                    __builtin_amdgcn_wave_barrier();
                    if (idx >= c)
                        chosen[idx + 1] = val;
                    __builtin_amdgcn_wave_barrier();
                }
                if (lane == 0)
                    chosen[c] = x + (uint32_t)c;
                __builtin_amdgcn_wave_barrier();
            }
            for (int32_t e = lane; e < s; e += kWave)
                put(e, src[chosen[e]]);
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
    }
}

// Registers per lane by fanout; above 256 positions the list's upkeep costs more than the binary search in LDS.  With
// independent draws only the one-register form is used (64 draws sorted across the lanes).  parts by the likely rows: by their bound
// the workgroups that have any were too few (hops of 7000 to 18000 rows, bound 65536: calls of 94 to 122 us now 73 to 108).
template <bool SET, bool REPLACE>
static void launch_nw_sample_wide(const Launch &L, const NwHop &a, const VSet &vs, int64_t tiles)
{
    const int64_t wanted = (int64_t)L.num_cu * 8, likely = a.rows_tune / kRowTile + a.k;
    int32_t parts = 1;
    while (parts < kRowTile / (kRowTile / kWave) && likely * parts < wanted)
        parts <<= 1;
    const dim3 block(kRowTile);
    if (a.s <= kWave)
        hipLaunchKernelGGL((nw_sample_wide_kernel<SET, REPLACE, 1>), dim3(grid_for(L, tiles * parts, 8)), block, 0, L.stream, a, vs, parts);
    else if (!REPLACE && a.s <= 2 * kWave)
        hipLaunchKernelGGL((nw_sample_wide_kernel<SET, REPLACE, REPLACE ? 0 : 2>), dim3(grid_for(L, tiles * parts, 8)), block, 0, L.stream, a, vs, parts);
    else if (!REPLACE && a.s <= 4 * kWave)
        hipLaunchKernelGGL((nw_sample_wide_kernel<SET, REPLACE, REPLACE ? 0 : 4>), dim3(grid_for(L, tiles * parts, 8)), block, 0, L.stream, a, vs, parts);
    else
        hipLaunchKernelGGL((nw_sample_wide_kernel<SET, REPLACE, 0>), dim3(grid_for(L, tiles * parts, 4)), block, 0, L.stream, a, vs, parts);
}

template <bool SET, bool REPLACE, bool SUM, bool DIES>
static void launch_nw_sample_lanes(const Launch &L, const NwHop &a, const VSet &vs, int grid)
{
    void (*const kernels[6])(NwHop, VSet) = {nw_sample_kernel<4, SET, REPLACE, SUM, DIES>,
                                             nw_sample_kernel<8, SET, REPLACE, SUM, DIES>,
                                             nw_sample_kernel<16, SET, REPLACE, SUM, DIES>,
                                             nw_sample_kernel<32, SET, REPLACE, SUM, DIES>,
                                             nw_sample_kernel<REPLACE ? 32 : 48, SET, REPLACE, SUM, DIES>,
                                             nw_sample_kernel<REPLACE ? 32 : 64, SET, REPLACE, SUM, DIES>};
    const int which = a.s <= 4 ? 0 : a.s <= 8 ? 1 : a.s <= 16 ? 2 : a.s <= 32 ? 3 : a.s <= 48 ? 4 : 5;
    hipLaunchKernelGGL(kernels[which], dim3(grid), dim3(kRowTile), 0, L.stream, a, vs);
}

// Fanouts of 33 .. 64 by one row per lane from this many rows or entries on.  A draw is two instructions per place then, for 64
// rows at once, where a row that has the wave to itself spends some ten on it; but with fewer rows most of the chip's waves have
// none, and rows that are copied whole take a lane as long as the others.  Whole calls on 2.4 M vertices, by lanes and by waves, us:
//   one hop, 8 minibatches       s = 33     s = 40     s = 48     s = 64
//   38 neighbours,  24576 rows   57,  62    60,  62    62,  63    79,  66
//                   40960        61,  69    64,  73    67,  74    84,  77
//                   65536        72,  90    74,  93    77,  94    88, 102
//   14 neighbours,  40960        62,  63    66,  65    69,  65    83,  65
//                   65536        67,  76    70,  75    74,  77    85,  78
//   two hops, the second one's million entries, 6 minibatches
//                   0.4 to 0.5  135, 132   138, 132   131, 122   147, 132
//                   0.7 to 0.8   96, 103   139, 137   149, 150    96,  87
//                   1.0 to 1.1  104, 113   118, 132   121, 124   120, 115
//                   1.4 to 1.5                        126, 140   135, 143
// Where the kernel also sets bits (few minibatches), by waves up to the 1.4 million: 0.8 million entries 109, 101, 1.4 million 145, 142.
// The rows and entries of later hops are what they are or were in the call before, not their bounds: 1024 seeds with (64, 64), 15000
// rows where k b s is 65536, took 114 us by lanes and take 100.  8 minibatches of 512, (40, 40), 51 neighbours: the second hop's
// sampling 76 -> 34 us by lanes, and it counts per segment, which saves 9 us more.
static bool wide_by_lanes(const NwHop &a, bool set)
{
    return a.rows_tune >= 65536 || a.entries_tune >= (a.s <= 48 && !set ? 15'000 * a.s : 1'400'000);
}
constexpr int32_t kMostSegmentsByDies = 128;
constexpr int64_t kMostStepBytes = 27 << 20;
template <bool SET, bool REPLACE>
static bool launch_nw_sample_impl(const Launch &L, const NwHop &a_in, const VSet &vs)
{
    NwHop a = a_in;
    const int64_t tiles = a.rows_bound / kRowTile + a.k;
    if (a.s > (!REPLACE && wide_by_lanes(a, SET) ? 64 : 32)) {
        a.seg_cnt = nullptr; // one row per wave: its workgroups walk the tiles in stacked order, across minibatches
        launch_nw_sample_wide<SET, REPLACE>(L, a, vs, tiles);
        return false;
    }
    // Four workgroups per compute unit: their 1024 rows hold more reads than the unit keeps in flight (about 92), and the
    // fewer rows are in progress on the chip, the narrower the part of A that the minibatches read at the same time: with
    // eight, it no longer fits the 256 MB last-level cache on the larger graphs.  Six where A's columns take four times that
    // cache at most, so that most of what several minibatches read is kept anyhow, and fanouts of up to 8 (above, five workgroups
    // fill LDS).  Last hop, stacked (by_dies below), by four and by six: 490 MB of columns 332 and 323 us, with own vertices 231 and
    // 212, with replacement 127 and 118; 5.3 GB (128 minibatches) 1185 and 1377 us, 6.4 GB 790 and 809.  Between, uniform graphs of 1 to 4 GB: 1 or 2 %
    // in six's favour, which is not worth what the larger skewed ones lose.
    const bool small_graph = a.A_nnz * (int64_t)sizeof(int32_t) <= (int64_t)1 << 30;
    int grid = grid_for(L, tiles, small_graph && a.s <= 8 ? 6 : 4);
    // counting per segment needs every workgroup to stay with one minibatch: tile v belongs to minibatch v % k,
    // so a grid that is a multiple of k does it
    if (!(a.seg_cnt && a.seg_C <= kMaxFusedSegments && a.k <= L.num_cu * 8))
        a.seg_cnt = nullptr;
    // By dies from one row for every two vertices on: then the minibatches' rows at the same place share lines.  Whole calls of
    // (15, 10, 5), stacked and by dies: 2.4 M vertices, rows / n 0.43 253 and 248 us, 0.86 368 and 351, 1.1 446 and 416, 2.3 719 and
    // 635 (the last hop's sampling 323 and 246); 4 M of 150 neighbours 0.46 484 and 482, 1.8 1224 and 1184; 0.5 M 0.65 125 and 118;
    // (15, 20) with 0.27 260 and 260; hops of few tiles, 100 x 400 seeds, (5, 15), of 0.2 M vertices 107 and 100; 20 x 600, (10, 10), of
    // 30 thousand 89 and 86.  Below that the second hop of 64 x 1024 seeds, 0.37, loses 5 us.
    // Counting per segment, a workgroup by dies leaves its counts after every tile: up to kMostSegmentsByDies of them, and from one row
    // for every eight vertices on, four with fanouts above 8 (20 M vertices, (10, 10, 10), 0.4 and more 1091 and 1034; a hop of ten with
    // 0.19, on 8.7 M, 288 and 298).  Calls of (15, 10, 5), 8.7 M vertices: 154 neighbours, 1.7 2452 and 2410, 0.8 1254 and 1244, 0.4 760
    // and 761; 53 neighbours, 1.1 1300 and 1168, 0.5 757 and 721; 12 neighbours, 0.44 562 and 543, 0.22 359 and 343; 20 M of 30
    // neighbours, 0.45 1184 and 1141, 0.2 710 and 700.
    // Of many minibatches with few tiles each a step spans more of the ids: up to kMostStepBytes of A's columns, so that the eight dies'
    // places fit the last-level cache together.  Last hop of (10, 10, 5), stacked and by dies: 8.7 M vertices of 154 neighbours, 200
    // minibatches (24 MB) 902 and 893 us, 256 (30) 892 and 939, 512 (58) 906 and 1063, 1000 (119) 937 and 1125; of 29 neighbours, 512 (17)
    // 430 and 401, 1000 (33) 433 and 450, 2000 (69) 500 and 541; of 7, 1000 (17) 151 and 144, 2000 (36) 165 and 187; 20 M of 21, 320 (26) 343
    // and 334, 430 (34) 365 and 354, 512 (40) 346 and 378, 1000 (81) 350 and 418.
    // With a table of segments, that is, where the sampled ids crowd a part of the id range, in stacked order: the die that has that part
    // has the rows of most entries, and the table is copied to LDS for every tile.  Ids by descending degree, stacked and by dies: 8.7 M
    // vertices, 154 neighbours, (8, 8, 8) 0.83 1920 and 2034, (6, 6, 6) 0.24 661 and 674; 53 neighbours, (8, 8, 8) 0.59 1174 and 1217,
    // (15, 10, 5) 0.27 544 and 564, 1.1 1509 and 1510; 12 neighbours, 0.48 685 and 713.
    // A workgroup by dies has one tile as a rule: those in progress then are neighbours, where workgroups that go on drift apart
    // (64 x 1024 seeds, 2.4 M vertices: two hops 305 us with six workgroups per compute unit that go on, 322 with four, 295 so;
    // independent draws, 32 x 777, are left going on: the call 333.3 so, 333.8 with a tile each).  But not where that is between 1.2 and 2
    // rounds of what the chip holds at a time: a second round that is half empty costs more than that.  0.5 M vertices of 78 neighbours, second
    // hop, going on and a tile each: 100 x 512 seeds, (10, 10, 5) (1.6 rounds), 39.4 and 43.9 us, 30 x 500, (40, 10) (1.7), 31.0 and 33.4;
    // 65 x 512, (10, 10) (1.1) 30.1 and 26.6, 130 x 512 (2.1) 46.3 and 43.5.
    const int64_t step_bytes = a.A_nnz * (int64_t)sizeof(int32_t) / std::max<int64_t>(a.rows_tune / a.k / kRowTile, 1);
    const bool counted_by_dies = !a.seg_tab && a.seg_C <= kMostSegmentsByDies && (a.s <= 8 ? 8 : 4) * a.rows_tune >= a.n && step_bytes <= kMostStepBytes;
    const bool by_dies = a.k >= kDies && (a.seg_cnt ? counted_by_dies : 2 * a.rows_tune >= a.n);
    const int64_t visits = likely_visits(a), at_a_time = (int64_t)L.num_cu * (a.s <= 8 ? 7 : a.s <= 16 ? 5 : a.s <= 32 ? 3 : 2); // (registers, LDS)
    if (by_dies && !REPLACE && (5 * visits <= 6 * at_a_time || visits >= 2 * at_a_time))
        grid = grid_for(L, visits, kOnePass);
    if (by_dies)
        grid = (grid + kDies - 1) / kDies * kDies;
    else if (a.seg_cnt)
        grid = std::max(grid / a.k, 1) * a.k;
    void (*const launch[2][2])(const Launch &, const NwHop &, const VSet &, int) = {
        {launch_nw_sample_lanes<SET, REPLACE, false, false>, launch_nw_sample_lanes<SET, REPLACE, false, true>},
        {launch_nw_sample_lanes<SET, REPLACE, true, false>, launch_nw_sample_lanes<SET, REPLACE, true, true>}};
    launch[a.sum_tiles ? 1 : 0][by_dies ? 1 : 0](L, a, vs, grid);
    return a.seg_cnt != nullptr;
}

bool launch_nw_sample(const Launch &L, const NwHop &a, const VSet &vs, bool set_bits)
{
    if (a.replace) {
        if (set_bits)
            return launch_nw_sample_impl<true, true>(L, a, vs);
        return launch_nw_sample_impl<false, true>(L, a, vs);
    }
    if (set_bits)
        return launch_nw_sample_impl<true, false>(L, a, vs);
    return launch_nw_sample_impl<false, false>(L, a, vs);
}

// ---------------------------------------------------------------------------------------------
// EXTRACT: "remove empty columns" -- the kept columns of a minibatch are its set vertices in
// ascending order, so a sampled vertex's local column is its rank in the vertex set:
// line_prefix[line] + set bits before it inside its 64-byte line.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void nw_relabel_kernel(NwHop a, VSet vs)
{
    const int64_t ntiles = a.mb_tileoff[a.k];
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int i = locate_segment(a.mb_tileoff, a.k, t);
        const uint32_t *__restrict__ words = vs.words + (int64_t)i * vs.nw;
        const uint32_t *__restrict__ prefix = vs.line_prefix + (int64_t)i * vs.nl;
        const int64_t e1 = a.tile_off[t + 1];
        for (int64_t e = a.tile_off[t] + threadIdx.x; e < e1; e += 256)
            a.out_col[e] = vset_rank_of(words, prefix, a.out_col[e]);
    }
}

// ---------------------------------------------------------------------------------------------
// Rows that carried their own vertex through EXTRACT as a trailing entry (so that it became a column
// and got a local index like any sampled vertex): the entry leaves the row again.  Row r loses one
// entry and every row before it one each, so its entries move r places down; the trailing entry is
// the row's own column.  One tile of kRowTile stacked rows per iteration, one entry per lane per
// step, the entry's row found in the tile's row offsets held in LDS.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kRowTile) void nw_strip_self_kernel(const int64_t *__restrict__ rowptr_in,
                                                                 const int32_t *__restrict__ col_in,
                                                                 const int64_t *__restrict__ rows_ptr,
                                                                 int64_t *__restrict__ rowptr_out,
                                                                 int32_t *__restrict__ col_out,
                                                                 int32_t *__restrict__ row_self,
                                                                 int64_t *__restrict__ nnz_slot)
{
    constexpr int kMapCap = kRowTile * 33; // entries of a tile whose rows hold at most 32 sampled vertices
    __shared__ int64_t off[kRowTile + 1];
    __shared__ uint8_t row_of[kMapCap];
    const int tid = threadIdx.x;
    const int64_t rows = *rows_ptr;
    const int64_t ntiles = (rows + kRowTile - 1) / kRowTile;
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int64_t r0 = t * kRowTile;
        const int nr = (int)(rows - r0 < kRowTile ? rows - r0 : kRowTile);
        const int64_t e0 = rowptr_in[r0];
        if (tid < nr) {
            const int64_t p = rowptr_in[r0 + tid];
            off[tid] = p - e0;
            rowptr_out[r0 + tid] = p - (r0 + tid);
        }
        if (tid == 0)
            off[nr] = rowptr_in[r0 + nr] - e0;
        __syncthreads();
        const int64_t span = off[nr];
        const bool mapped = span <= kMapCap; // the usual case: every row writes its index over its entries
        if (mapped && tid < nr) {
            const int32_t b = (int32_t)off[tid], e = (int32_t)off[tid + 1];
            for (int32_t q = b; q < e; ++q)
                row_of[q] = (uint8_t)tid;
        }
        if (mapped)
            __syncthreads();
        for (int64_t e = tid; e < span; e += kRowTile) {
            int lo;
            if (mapped) {
                lo = row_of[e];
            } else { // last row with off[row] <= e (rows are never empty: each has its own entry)
                lo = 0;
                int hi = nr;
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (off[mid] <= e)
                        lo = mid;
                    else
                        hi = mid;
                }
            }
            const int32_t g = col_in[e0 + e];
            if (e == off[lo + 1] - 1)
                row_self[r0 + lo] = g;
            else
                col_out[e0 + e - (r0 + lo)] = g;
        }
        __syncthreads();
    }
    if (blockIdx.x == 0 && tid == 0) {
        const int64_t total = rowptr_in[rows];
        rowptr_out[rows] = total - rows;
        *nnz_slot = total - rows;
    }
}

void launch_nw_strip_self(const Launch &L, const int64_t *rowptr_in, const int32_t *col_in, const int64_t *rows,
                          int64_t rows_bound, int64_t *rowptr_out, int32_t *col_out, int32_t *row_self,
                          int64_t *nnz_slot)
{
    const int64_t tiles = rows_bound / kRowTile + 1;
    hipLaunchKernelGGL(nw_strip_self_kernel, dim3(grid_for(L, tiles, 8)), dim3(kRowTile), 0, L.stream, rowptr_in,
                       col_in, rows, rowptr_out, col_out, row_self, nnz_slot);
}

void launch_nw_relabel(const Launch &L, const NwHop &a, const VSet &vs)
{
    const int64_t tiles = a.rows_bound / kRowTile + a.k;
    hipLaunchKernelGGL(nw_relabel_kernel, dim3(grid_for(L, tiles, 16)), dim3(256), 0, L.stream, a, vs);
}

} // namespace bms
