// EXTRACT for the node-wise sampler, main path (Sec. 4.1.3: "remove empty columns"): every
// minibatch's sampled ids are cut into C id ranges ("segments") small enough to be ranked inside
// LDS, so that all random accesses of the dedup happen in LDS and global memory only sees
// coalesced traffic.  Positions never travel with the ids: the cut remembers, per position, its place
// in the tile's ids sorted by segment, and per (tile, segment) where that run went, so the ranks come
// back along the same runs.  All kernels run on every compute unit, whatever the
// number of minibatches.
//
//   count    per tile of 8192 positions: LDS histogram over the C segments -> global counts
//   scan     per minibatch: segment offsets; segments too long for one workgroup are listed for the
//            bitmap kernel; raises the fallback flag when a segment fits neither (ids crowded into a
//            narrow range) -- then these kernels do nothing and the per-minibatch kernel of
//            kernels_dedup.hip does the hop instead
//   split    per tile: counting sort by segment in LDS, every segment's run of ids appended to the
//            segment with wide stores; per position its place in the tile's order; per (tile, segment)
//            where the run went
//   rank     per (minibatch, segment): a workgroup counts the segment's ids into buckets of about
//            one id (LDS), every id compares itself with the few ids of its bucket, head bits and a
//            popcount prefix give every id its rank among the segment's distinct ids; the distinct
//            ids are written in rank order at the head of the segment's slots
//   bitmap   the listed segments: rank = set bits below the id in a bitmap of the segment's id range
//   base     per minibatch: scan of the segments' distinct counts
//   un-split per tile: the runs' ranks read back with wide loads, base of the segment added in LDS, read
//            from there by position, written out as the tile's local column indices
#include "bms_device.h"
#include "bms_internal.h"

#include <algorithm>

namespace bms {

static_assert(kCutTile <= 1 << 16, "places of the cut in 16 bits");

// Tiles of a minibatch's N positions, which begin at e0 of the stacked columns: all but the first one begin at a memory line (of an
// array that does), so that a tile's columns are read and written by whole lines.
__device__ inline int64_t cut_tiles(int64_t e0, int64_t N)
{
    return N ? (N + (e0 & (kLineEntries - 1)) + kCutTile - 1) / kCutTile : 0;
}
__device__ inline void cut_tile(int64_t e0, uint32_t N, uint32_t x, uint32_t &j0, uint32_t &jend) // tile x: positions j0 .. jend
{
    const uint32_t head = (uint32_t)e0 & (kLineEntries - 1);
    j0 = x ? x * kCutTile - head : 0;
    jend = (uint32_t)min<uint64_t>((uint64_t)(x + 1) * kCutTile - head, N);
}

// The table of segments of unequal width, copied to LDS by the kernels that look ids up (tab_l: kMaxCells + 1 entries).
__device__ inline void load_seg_table(const DedupArgs &a, uint16_t *tab_l, int nthreads)
{
    if (a.tab == nullptr)
        return;
    for (int x = threadIdx.x; x <= kMaxCells; x += nthreads)
        tab_l[x] = a.tab[x];
    __syncthreads();
}
__device__ inline uint32_t seg_of(const DedupArgs &a, const uint16_t *tab_l, uint32_t id)
{
    return a.tab ? (uint32_t)tab_l[id >> a.fshift] : id >> a.cshift;
}
// first id of segment c and log2 (rounded up) of the number of ids it spans
__device__ inline void seg_range(const DedupArgs &a, uint32_t c, uint32_t &id0, int &wbits)
{
    if (a.tab) {
        const uint32_t f0 = a.seg_first[c], width = (a.seg_first[c + 1] - f0) << a.fshift;
        id0 = f0 << a.fshift;
        wbits = width <= 1u ? 0 : 32 - __clz(width - 1u);
    } else {
        id0 = c << a.cshift;
        wbits = a.cshift;
    }
}

template <int TILE, int NT>
__global__ __launch_bounds__(NT) void dd_count_kernel(DedupArgs a, const int64_t *__restrict__ tileoff)
{
    __shared__ uint32_t hist[kMaxSegments];
    __shared__ uint16_t tab_l[kMaxCells + 1];
    const int tid = threadIdx.x;
    load_seg_table(a, tab_l, NT);
    const int64_t ntiles = tileoff[a.k];
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int i = locate_segment(tileoff, a.k, t);
        const int64_t e0 = a.mb_edgeoff[i];
        const uint32_t N = (uint32_t)(a.mb_edgeoff[i + 1] - e0);
        uint32_t j0, jend;
        cut_tile(e0, N, (uint32_t)(t - tileoff[i]), j0, jend);
        const int32_t *__restrict__ col = a.col + e0;
        for (int c = tid; c < a.C; c += NT)
            hist[c] = 0;
        __syncthreads();
        uint32_t g[TILE / NT];
#pragma unroll
        for (int q = 0; q < TILE / NT; ++q) {
            const uint32_t j = j0 + q * NT + tid;
            g[q] = j < jend ? (uint32_t)col[j] : 0xFFFFFFFFu;
        }
#pragma unroll
        for (int q = 0; q < TILE / NT; ++q)
            if (g[q] != 0xFFFFFFFFu)
                atomicAdd(&hist[seg_of(a, tab_l, g[q])], 1u);
        __syncthreads();
        for (int c = tid; c < a.C; c += NT)
            if (hist[c])
                atomicAdd(&a.seg_cnt[(int64_t)i * a.C + c], hist[c]);
        __syncthreads();
    }
}

// appends `value` of every lane with `flag` to a list in global memory: one atomic per wave
__device__ inline void wave_append(uint32_t *__restrict__ list, uint32_t *__restrict__ count, bool flag, uint32_t value)
{
    const unsigned long long mask = __ballot(flag);
    if (mask == 0)
        return;
    const int lane = threadIdx.x & (kWave - 1);
    const int leader = __ffsll((long long)mask) - 1;
    uint32_t base = 0;
    if (lane == leader)
        base = atomicAdd(count, (uint32_t)__popcll(mask));
    base = __shfl(base, leader, kWave);
    if (flag)
        list[base + __popcll(mask & ((1ull << lane) - 1ull))] = value;
}

constexpr int kRankCapFwd = 4096; // = kRankCap (defined with the ranking kernel below)

// one workgroup per minibatch: seg_off = exclusive scan of the counts (C+1 entries), cursors zeroed
__device__ inline void seg_scan_block(const DedupArgs &a, int i, uint32_t *smem, uint32_t &carry_s)
{
    const int tid = threadIdx.x;
    const uint32_t *__restrict__ cnt = a.seg_cnt + (int64_t)i * a.C;
    uint32_t *__restrict__ off = a.seg_off + (int64_t)i * (a.C + 1);
    if (tid == 0)
        carry_s = 0;
    __syncthreads();
    bool too_big = false;
    for (int base = 0; base < a.C; base += 256) {
        const int c = base + tid;
        const uint32_t v = c < a.C ? cnt[c] : 0u;
        // too many entries for one workgroup of the ranking kernel: listed for the bitmap kernel, which holds the
        // segment's id range as bits in LDS; a segment wider or fuller than that kernel takes sends the hop to the
        // per-minibatch kernel
        const bool big = !a.by_bitmap && v > (uint32_t)kRankCapFwd;
        if (big || v > (uint32_t)kSegCap) {
            uint32_t id0;
            int wbits;
            seg_range(a, (uint32_t)c, id0, wbits);
            too_big |= v > (uint32_t)kSegCap || wbits > a.wbits_max;
        }
        wave_append(a.big_list, a.big_count, big && v <= (uint32_t)kSegCap, (uint32_t)(i * a.C + c));
        uint32_t total;
        const uint32_t ex = block_exclusive_scan<uint32_t, 256>(v, smem, total);
        const uint32_t carry = carry_s;
        if (c < a.C) {
            off[c] = carry + ex;
            a.seg_cursor[(int64_t)i * a.C + c] = 0;
        }
        __syncthreads();
        if (tid == 0)
            carry_s = carry + total;
        __syncthreads();
    }
    if (tid == 0)
        off[a.C] = carry_s;
    if (too_big)
        atomicOr(a.fallback, 1);
}

// Planning of a hop's EXTRACT in one launch.  Workgroup k: first entry of every minibatch in the stacked column
// array (mb_edgeoff[i] = rowptr[mb_rowoff[i]]) and the tiles of the cut (tiles never straddle minibatches).
// Workgroups 0..k-1 (only with `scan`, i.e. when the counts per segment are there already): the segment offsets
// of minibatch i.
__global__ __launch_bounds__(256) void dd_plan_kernel(DedupArgs a, const int64_t *__restrict__ out_rowptr,
                                                      const int64_t *__restrict__ mb_rowoff, int scan)
{
    __shared__ uint32_t smem[4];
    __shared__ uint32_t carry_s;
    __shared__ int64_t smem64[4];
    __shared__ int64_t carry64_s;
    if ((int)blockIdx.x < a.k) {
        if (scan)
            seg_scan_block(a, blockIdx.x, smem, carry_s);
        return;
    }
    const int tid = threadIdx.x;
    if (tid == 0)
        carry64_s = 0;
    __syncthreads();
    for (int32_t base = 0; base < a.k; base += 256) {
        const int32_t i = base + tid;
        int64_t cnt = 0;
        if (i < a.k) {
            const int64_t e0 = out_rowptr[mb_rowoff[i]], e1 = out_rowptr[mb_rowoff[i + 1]];
            a.mb_edgeoff[i] = e0;
            if (i == a.k - 1)
                a.mb_edgeoff[a.k] = e1;
            cnt = cut_tiles(e0, e1 - e0);
        }
        int64_t total;
        const int64_t ex = block_exclusive_scan<int64_t, 256>(cnt, smem64, total);
        const int64_t carry = carry64_s;
        if (i < a.k)
            a.big_tileoff[i] = carry + ex;
        __syncthreads();
        if (tid == 0)
            carry64_s = carry + total;
        __syncthreads();
    }
    if (tid == 0)
        a.big_tileoff[a.k] = carry64_s;
}

__global__ __launch_bounds__(256) void dd_seg_scan_kernel(DedupArgs a)
{
    __shared__ uint32_t smem[4];
    __shared__ uint32_t carry_s;
    seg_scan_block(a, blockIdx.x, smem, carry_s);
}

// TILE positions per workgroup step, NT threads.  The larger the tile, the longer the run every segment gets
// in one step (a step's ids spread over all C segments), i.e. the wider the stores.  Three workgroups share a compute unit, with 70
// registers (four, in 64, spill: 0.152 ms for 0.133).  Two hops of 256 x 1024 seeds, (15, 10, 5), 111 M vertices, 58 M entries: 0.160 ms with a
// thousand workgroups that go from tile to tile, 0.143 with a tile each, 0.133 without a mask per id in whole tiles and with the
// table of segments as a kernel of its own; of 128 on 8.7 M, 86 M entries: 0.238, 0.203 and 0.190.
constexpr int kSplitThreads = 512;
template <int TILE, int NT, bool TAB>
__global__ __launch_bounds__(NT, 6) void dd_split_kernel(DedupArgs a, const int64_t *__restrict__ tileoff)
{
    // stage[TILE]; then 3 C words: per-segment count, start in the tile, start in global - start in the tile; then the table of
    // segments, if there is one (TAB: a.tab; without it the segment of an id is a shift, and nothing is copied first)
    extern __shared__ uint32_t split_lds[];
    __shared__ uint32_t smem[NT / kWave];
    __shared__ uint32_t carry_s;
    if (*a.fallback)
        return;
    uint32_t *stage = split_lds;
    uint32_t *cnt = split_lds + TILE, *off = cnt + a.C, *gpos = cnt + 2 * a.C;
    uint16_t *tab_l = reinterpret_cast<uint16_t *>(cnt + 3 * a.C);
    if (TAB)
        load_seg_table(a, tab_l, NT);
    const int shift = TAB ? a.fshift : a.cshift;
    auto segment = [&](uint32_t id) { return TAB ? (uint32_t)tab_l[id >> shift] : id >> shift; };
    const int64_t ntiles = uniform_load(tileoff + a.k);
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid)); // (places: computed anew for every tile, not kept in registers)
        const int i = locate_uniform(tileoff, a.k, t);
        const int64_t e0 = uniform_load(a.mb_edgeoff + i);
        const uint32_t N = (uint32_t)(uniform_load(a.mb_edgeoff + i + 1) - e0);
        uint32_t j0, jend;
        cut_tile(e0, N, (uint32_t)(t - uniform_load(tileoff + i)), j0, jend);
        const int n = (int)scalar(jend - j0), left = n - tid;
        const int32_t *__restrict__ col = a.col + scalar(e0 + j0);
        uint16_t *__restrict__ loc = a.loc + scalar(e0 + j0);
        uint32_t id[TILE / NT]; // (< 2^31)
        uint32_t place[TILE / NT]; // in the tile's run for the segment
#pragma unroll
        for (int q = 0; q < TILE / NT; ++q) {
            id[q] = left > q * NT ? (uint32_t)(col + q * NT)[tid] : 0;
            place[q] = 0;
        }
        for (int c = tid; c < a.C; c += NT)
            cnt[c] = 0;
        if (tid == 0)
            carry_s = 0;
        __syncthreads();
        // (whole tiles without a mask per id)
        auto each = [&](auto body) {
            if (n == TILE) {
#pragma unroll
                for (int q = 0; q < TILE / NT; ++q)
                    body(q);
            } else {
#pragma unroll
                for (int q = 0; q < TILE / NT; ++q)
                    if (left > q * NT)
                        body(q);
            }
        };
        each([&](int q) { place[q] = atomicAdd(&cnt[segment(id[q])], 1u); });
        __syncthreads();
        uint32_t *__restrict__ run_gpos = a.run_gpos + t * a.C, *__restrict__ run_cnt = a.run_cnt + t * a.C;
        for (int base = 0; base < a.C; base += NT) {
            const int c = base + tid;
            const uint32_t v = c < a.C ? cnt[c] : 0u;
            uint32_t total;
            const uint32_t ex = block_exclusive_scan<uint32_t, NT>(v, smem, total);
            const uint32_t carry = carry_s;
            if (c < a.C) {
                off[c] = carry + ex;
                uint32_t g = 0;
                if (v)
                    g = a.seg_off[(int64_t)i * (a.C + 1) + c] + atomicAdd(&a.seg_cursor[(int64_t)i * a.C + c], v);
                gpos[c] = g - (carry + ex); // start in global - start in the tile
                run_gpos[c] = g;
                run_cnt[c] = v;
            }
            __syncthreads();
            if (tid == 0)
                carry_s = carry + total;
            __syncthreads();
        }
        each([&](int q) {
            const uint32_t at = off[segment(id[q])] + place[q];
            stage[at] = id[q];
            (loc + q * NT)[tid] = (uint16_t)at;
        });
        __syncthreads();
        uint32_t *__restrict__ ids_seg = a.ids_seg + e0;
        each([&](int q) {
            const uint32_t g = (stage + q * NT)[tid];
            ids_seg[gpos[segment(g)] + (uint32_t)(q * NT + tid)] = g;
        });
        __syncthreads();
    }
}

// One workgroup per (minibatch, segment) of at most kRankCap ids: ranks by counting, no sorting network.
// Every thread keeps its ids (slot j = q NT + tid) in registers through all steps.
//   1  the ids are counted into up to 4096 buckets by their leading bits (about one id per bucket)
//   2  exclusive scan of the bucket sizes (every wave a contiguous part, 16 bytes per lane and access);
//      a bucket of more than kRankMaxInBucket ids (one id sampled by many rows, ids crowded into a narrow range)
//      hands the segment to the bitmap kernel, or the hop to the per-minibatch kernel when the segment is too
//      wide for that
//   3  every id goes to its bucket's place in LDS
//   4  every id looks at the few ids of its bucket and sets bit (bucket start + smaller ones) = the place of its run of equal
//      ids in ascending order
//   5  popcount prefix over the bits: the rank of an id among the distinct ones = runs before its own
//   6  ranks leave in slot order; the ids go to their rank, copied out as the distinct ids
// A chain of dependent LDS steps, so what counts is how many workgroups share a compute unit.  256 x 240 k ids of 111 M: 343 us with
// two, 296 with three that went from one segment to the next and fetched its ids ahead (80 registers).  A workgroup per segment
// needs no loop, whose carried values and places cost half of the registers (45 without), so that four share a unit, and nobody waits
// for a segment's stores: two hops of that call 384 us so far, 349 started per segment with the loop, 280 without.  About 13 LDS
// accesses per id bound it.
constexpr int kRankCap = 4096;    // ids of a segment that one workgroup of the ranking kernel takes
constexpr int kRankThreads = 512;
constexpr int kRankBucketBits = 12; // at most 4096 buckets
constexpr int kRankMaxInBucket = 32;
static_assert(kRankCap == kRankCapFwd, "segment capacity out of step");

__global__ __launch_bounds__(kRankThreads, 8) void dd_rank_kernel(DedupArgs a)
{
    constexpr int NT = kRankThreads, NW = NT / kWave, PER = kRankCap / NT, NB = 1 << kRankBucketBits;
    __shared__ uint4 cnt4[NB / 4 + 1];           // bucket sizes, then bucket starts; start[nb] = m
    __shared__ uint32_t sorted[kRankCap + 3];    // ids by bucket (relative to the segment's first id); then the distinct ones
    __shared__ uint32_t hbits[kRankCap / 32], hpre[kRankCap / 32];
    __shared__ uint32_t wtot[NW];
    uint32_t *cnt = reinterpret_cast<uint32_t *>(cnt4);
    if (*a.fallback)
        return;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const uint32_t cseg = blockIdx.y;
    const int64_t i = blockIdx.x; // workgroups that run at the same time take segments of different minibatches
    const int64_t sg = i * a.C + cseg;
    const uint32_t s0 = uniform_load(a.seg_off + i * (a.C + 1) + cseg), m = uniform_load(a.seg_off + i * (a.C + 1) + cseg + 1) - s0;
    const int64_t e0 = uniform_load(a.mb_edgeoff + i);
    if (m > (uint32_t)kRankCap || m == 0) { // listed for the bitmap kernel by the scan, or empty
        if (m == 0 && tid == 0)
            a.seg_cnt[sg] = 0;
        return;
    }
    uint32_t key[PER]; // slot j = q NT + tid, unused slots all ones
    const uint32_t *__restrict__ ids = a.ids_seg + e0 + s0;
#pragma unroll
    for (int q = 0; q < PER; ++q)
        key[q] = (uint32_t)(q * NT + tid) < m ? ids[q * NT + tid] : 0xFFFFFFFFu;
    uint32_t id0;
    int wbits;
    seg_range(a, cseg, id0, wbits);
    // buckets: a power of two >= m, 512..4096, no more than the segment has ids
    int nbits = 32 - __clz(m - 1u); // ceil(log2 m); m = 1: __clz(0) = 32
    if (m == 1u || nbits < 9)
        nbits = 9;
    if (nbits > kRankBucketBits)
        nbits = kRankBucketBits;
    if (nbits > wbits)
        nbits = wbits;
    const int bshift = wbits - nbits;
    const int nb = 1 << nbits;
    const int nqd = nb >= 4 ? nb / 4 : 1;                  // 16-byte quads of counters
    const int qw = (nqd + NW - 1) / NW;                    // per wave
    const int its = (qw + kWave - 1) / kWave;              // per lane: 1 or 2
    for (int qd = tid; qd < nqd; qd += NT)
        cnt4[qd] = make_uint4(0, 0, 0, 0);
    for (uint32_t x = tid; x < (m + 31u) / 32u; x += NT)
        hbits[x] = 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (key[q] != 0xFFFFFFFFu)
            key[q] -= id0;
    uint32_t at[PER]; // slot in the bucket; then the bucket's start, size (from bit 13) and the slot; from step 4 on: place of the id's run
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (key[q] != 0xFFFFFFFFu)
            at[q] = atomicAdd(&cnt[key[q] >> bshift], 1u);
    __syncthreads();
    // exclusive scan of the bucket sizes, in place
    uint4 cv[2];
    uint32_t inc[2], mine[2];
    uint32_t wave_total = 0;
    bool crowded = false;
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        cv[it] = make_uint4(0, 0, 0, 0);
        mine[it] = inc[it] = 0;
        if (it < its) {
            const int lq = it * kWave + lane; // quad inside this wave's part
            if (lq < qw && wave * qw + lq < nqd)
                cv[it] = cnt4[wave * qw + lq];
            crowded |= cv[it].x > (uint32_t)kRankMaxInBucket || cv[it].y > (uint32_t)kRankMaxInBucket ||
                       cv[it].z > (uint32_t)kRankMaxInBucket || cv[it].w > (uint32_t)kRankMaxInBucket;
            mine[it] = cv[it].x + cv[it].y + cv[it].z + cv[it].w;
            inc[it] = wave_inclusive_scan_dpp(mine[it]) + wave_total;
            wave_total = (uint32_t)__builtin_amdgcn_readlane((int)inc[it], kWave - 1);
        }
    }
    if (lane == 0)
        wtot[wave] = wave_total;
    if (__syncthreads_or(crowded)) { // uniform for the workgroup
        if (tid == 0) {
            if (wbits <= a.wbits_max)
                a.big_list[atomicAdd(a.big_count, 1u)] = (uint32_t)sg;
            else
                atomicOr(a.fallback, 1);
        }
        return;
    }
    uint32_t run = 0;
#pragma unroll
    for (int w2 = 0; w2 < NW; ++w2)
        run += w2 < wave ? wtot[w2] : 0u;
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        if (it < its) {
            const int lq = it * kWave + lane;
            if (lq < qw && wave * qw + lq < nqd) {
                const uint32_t s = run + inc[it] - mine[it];
                cnt4[wave * qw + lq] = make_uint4(s, s + cv[it].x, s + cv[it].x + cv[it].y, s + cv[it].x + cv[it].y + cv[it].z);
            }
        }
    }
    if (tid == 0)
        cnt[nb] = m;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (key[q] != 0xFFFFFFFFu) {
            const uint32_t bucket = key[q] >> bshift, bs = cnt[bucket], be = cnt[bucket + 1u];
            sorted[bs + at[q]] = key[q];
            at[q] = at[q] << 19 | (be - bs) << 13 | bs;
        }
    if (tid < 3)
        sorted[m + tid] = 0xFFFFFFFFu; // (step 4 reads that far)
    __syncthreads();
    // place of every id's run of equal ids in ascending order; heads
    if (bshift == 0) { // one id per bucket: the run is the bucket
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (key[q] != 0xFFFFFFFFu) {
                const uint32_t p = at[q] & 8191u;
                if (at[q] >> 19 == 0)
                    atomicOr(&hbits[p >> 5], 1u << (p & 31u));
                at[q] = p;
            }
    } else {
        // the ids after a bucket are larger than its own: four reads each, of two ids at a time, whatever the bucket's size
#pragma unroll
        for (int q0 = 0; q0 < PER; q0 += 2) {
            uint32_t o[2][4];
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    o[u][t] = sorted[(key[q0 + u] != 0xFFFFFFFFu ? at[q0 + u] & 8191u : 0u) + t];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int q = q0 + u;
                if (key[q] == 0xFFFFFFFFu)
                    continue;
                const uint32_t bs = at[q] & 8191u, n = (at[q] >> 13) & 63u;
                uint32_t p = bs;
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    p += o[u][t] < key[q] ? 1u : 0u;
                for (uint32_t t = 4; t < n; ++t)
                    p += sorted[bs + t] < key[q] ? 1u : 0u;
                atomicOr(&hbits[p >> 5], 1u << (p & 31u));
                at[q] = p;
            }
        }
    }
    __syncthreads();
    const uint32_t nwd = (m + 31u) / 32u; // <= 128 words of head bits
    if (wave == 0) {
        uint32_t carry = 0;
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const uint32_t x = it * kWave + lane;
            const uint32_t pcw = x < nwd ? __popc(hbits[x]) : 0u;
            const uint32_t in2 = wave_inclusive_scan_dpp(pcw) + carry;
            if (x < nwd)
                hpre[x] = in2 - pcw;
            carry = (uint32_t)__builtin_amdgcn_readlane((int)in2, kWave - 1);
        }
        if (lane == 0) {
            wtot[0] = carry;
            a.seg_cnt[sg] = carry;
        }
    }
    __syncthreads();
    const uint32_t cnt_distinct = wtot[0];
    uint16_t *__restrict__ ranks = a.ranks + e0 + s0;
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (key[q] != 0xFFFFFFFFu) {
            const uint32_t p = at[q];
            const uint32_t r = hpre[p >> 5] + __popc(hbits[p >> 5] & ((1u << (p & 31u)) - 1u));
            ranks[q * NT + tid] = (uint16_t)r;
            sorted[r] = key[q]; // every id has been looked at (step 4): their place now takes the distinct ones
        }
    __syncthreads();
    uint32_t *__restrict__ uids = a.uids + e0 + s0;
    for (uint32_t r = tid; r < cnt_distinct; r += NT)
        uids[r] = id0 + sorted[r];
}

// Ranking through a bitmap of the segment's id range in LDS (2^cshift bits, at most 128 KB): no sort.  The rank
// of an id among the segment's distinct ids is the number of set bits below it.  Work per segment = one pass over the bitmap
// (16 bytes per lane and access, no bank conflicts) + a few operations per id, whatever the ids' multiplicities; a segment may
// hold up to kSegCap ids (a rank has 16 bits).  LISTED = false: every segment of the hop (hops whose ids are dense enough that
// the pass over the bitmap costs less than sorting); LISTED = true: the segments that the sorting kernel handed over.
//   1  the ids' bits are set (LDS atomics); the first kBmKeep ids of every thread stay in registers
//   2  every wave owns a contiguous part of the bitmap, in "quads" of 128 bits, quad it*64 + lane of the part in
//      iteration it: popcounts, wave totals -> set bits before the wave's part; running count before every quad
//      (16 bits, kept in LDS)
//   3  rank of an id = count before its quad + set bits below it inside the quad; every id goes to its rank's place in LDS
//      (equal ids to the same one), from where the distinct ids leave in order
//   4  LISTED, where a workgroup may have several segments: the bitmap is cleared again, word by word through the ids when they are
//      few, else as a whole
// What bounds it is latency: trips to memory for ids that are not in registers, and, before step 3 did it, the stores of the
// distinct ids straight from the bitmap, scattered over a wave's lanes (128 x 586 k ids of 8.7 M: 475 us so, 262 us without).
// Two workgroups share a compute unit, which leaves 64 registers: enough as long as what the lanes have in common is in scalar
// ones, and a workgroup has one segment (282 us for the two hops when it could have several, 255 so).  With a segment's place and length in every lane 14 registers went to memory and back, as many bytes again as the ids
// themselves: the last two hops of 128 x 1024 seeds, (15, 10, 5), took 373 us so and 281 us without.
constexpr int kBmThreads = 1024;
constexpr int kBmWaves = kBmThreads / kWave;
constexpr int kBmKeep = 10; // ids per thread kept in registers between the passes (segments up to 10240 ids)
constexpr int kBmIts = 8;   // quads per lane: 16 waves x 64 lanes x 8 quads x 128 bits = 2^20 bits
constexpr int kBmPlaces = 10240; // distinct ids that go through LDS, where it has room for them
static_assert(kBmWaves * kWave * kBmIts * 128 == (1 << kMaxBitmapShift), "bitmap geometry out of step");
static uint32_t bm_quads(int cshift)
{
    uint32_t quads = (uint32_t)(((size_t)1 << cshift) / 128);
    return quads < (uint32_t)(kBmWaves * kWave) ? (uint32_t)(kBmWaves * kWave) : quads; // every lane owns at least one quad
}
// places for distinct ids beside the bitmap: all of kBmPlaces as long as two workgroups share a compute unit
static int bm_places(int cshift) { return (size_t)bm_quads(cshift) * 18 + (size_t)kBmPlaces * 4 <= 78 * 1024 ? kBmPlaces : 0; }
size_t dd_bitmap_lds_bytes(int cshift)
{
    return (size_t)bm_quads(cshift) * 18 + (size_t)bm_places(cshift) * 4;
}

template <bool LISTED>
__global__ __launch_bounds__(kBmThreads, 8) void dd_bitmap_kernel(DedupArgs a, uint32_t places)
{
    extern __shared__ uint4 bm_lds[]; // quads, then `places` ids, then one 16-bit running count per quad
    __shared__ uint32_t wtot[kBmWaves];
    if (*a.fallback || a.wbits_max > kMaxBitmapShift)
        return;
    int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    uint32_t nq = (1u << a.wbits_max) / 128u;
    if (nq < (uint32_t)(kBmWaves * kWave))
        nq = kBmWaves * kWave;
    const int its = (int)(nq / (kBmWaves * kWave)); // quads per lane: 1, 2, 4 or 8
    uint4 *quads = bm_lds;
    uint32_t *words = reinterpret_cast<uint32_t *>(bm_lds);
    uint32_t *place = reinterpret_cast<uint32_t *>(bm_lds + nq);
    uint16_t *qpre = reinterpret_cast<uint16_t *>(place + places);
    const uint32_t q_wave = (uint32_t)wave * (uint32_t)(its * kWave); // first quad of this wave's part
    const uint32_t nwork = LISTED ? *a.big_count : 0u;
    if (LISTED && blockIdx.x >= nwork)
        return; // usually nothing is listed
    for (int it = 0; it < its; ++it)
        quads[q_wave + it * kWave + lane] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    // where a segment lies; the first ids of a listed one are fetched while the segment before it is worked on
    struct Seg {
        int64_t e0;
        uint32_t sg, s0, m, id0;
    };
    auto locate = [&](uint32_t x, Seg &g) {
        g.m = g.s0 = g.id0 = g.sg = 0;
        g.e0 = 0;
        if (LISTED && x >= nwork)
            return;
        uint32_t i = blockIdx.x, c = blockIdx.y; // workgroups that run at the same time take segments of different minibatches
        g.sg = i * (uint32_t)a.C + c;            // (fits: the list holds segments in 32 bits)
        if (LISTED) {
            g.sg = scalar(a.big_list[x]);
            i = g.sg / (uint32_t)a.C;
            c = g.sg % (uint32_t)a.C;
        }
        const uint32_t *__restrict__ soff = a.seg_off + (int64_t)i * (a.C + 1);
        int wbits;
        seg_range(a, c, g.id0, wbits);
        // the same in every lane: kept in scalar registers
        g.e0 = scalar(a.mb_edgeoff[i]);
        g.s0 = scalar(soff[c]);
        g.m = scalar(soff[c + 1]) - g.s0;
        g.id0 = scalar(g.id0);
    };
    auto fetch = [&](const Seg &g, uint32_t (&id)[kBmKeep]) { // relative to the segment's first id
        const uint32_t *__restrict__ ids = a.ids_seg + g.e0 + g.s0;
        uint32_t t = (uint32_t)tid;
        asm volatile("" : "+v"(t)); // (places of the loads: computed here, not kept in registers)
#pragma unroll
        for (int q = 0; q < kBmKeep; ++q)
            id[q] = q * kBmThreads + t < g.m ? ids[q * kBmThreads + t] : 0xFFFFFFFFu;
    };
    Seg cur, nxt;
    uint32_t keep[kBmKeep], next[kBmKeep];
    locate(blockIdx.x, cur);
    fetch(cur, next);
    for (uint32_t x = blockIdx.x; !LISTED || x < nwork; x += gridDim.x, cur = nxt) {
        if (LISTED) {
            asm volatile("" : "+v"(tid), "+v"(lane)); // (places: computed anew for every segment, not kept in registers)
            locate(x + gridDim.x, nxt);
        }
        const uint32_t m = cur.m, id0 = cur.id0;
#pragma unroll
        for (int q = 0; q < kBmKeep; ++q)
            keep[q] = next[q] == 0xFFFFFFFFu ? next[q] : next[q] - id0;
        if (m == 0) {
            if (tid == 0)
                a.seg_cnt[cur.sg] = 0;
            if (!LISTED)
                return;
            fetch(nxt, next);
            continue;
        }
        const uint32_t *__restrict__ ids = a.ids_seg + cur.e0 + cur.s0;
        uint16_t *__restrict__ ranks = a.ranks + cur.e0 + cur.s0;
        uint32_t *__restrict__ uids = a.uids + cur.e0 + cur.s0;
        // 1: set bits
#pragma unroll
        for (int q = 0; q < kBmKeep; ++q)
            if (keep[q] != 0xFFFFFFFFu)
                atomicOr(&words[keep[q] >> 5], 1u << (keep[q] & 31u));
        for (uint32_t j = kBmKeep * kBmThreads + tid; j < m; j += kBmThreads) {
            const uint32_t b = ids[j] - id0;
            atomicOr(&words[b >> 5], 1u << (b & 31u));
        }
        __syncthreads();
        if (LISTED)
            fetch(nxt, next);
        // 2: counts before every quad
        uint32_t inc[kBmIts];
        uint32_t wave_total = 0;
#pragma unroll
        for (int it = 0; it < kBmIts; ++it) {
            inc[it] = 0;
            if (it < its) {
                const uint4 qv = quads[q_wave + it * kWave + lane];
                const uint32_t pc = __popc(qv.x) + __popc(qv.y) + __popc(qv.z) + __popc(qv.w);
                const uint32_t upto = wave_inclusive_scan_dpp(pc) + wave_total; // set bits of this wave's part up to this quad
                inc[it] = upto - pc;
                wave_total = (uint32_t)__builtin_amdgcn_readlane((int)upto, kWave - 1);
            }
        }
        if (lane == 0)
            wtot[wave] = wave_total;
        __syncthreads();
        uint32_t run = 0, cnt = 0; // set bits before this wave's part; in the whole bitmap
#pragma unroll
        for (int w = 0; w < kBmWaves; ++w) {
            const uint32_t t = wtot[w];
            run += w < wave ? t : 0u;
            cnt += t;
        }
#pragma unroll
        for (int it = 0; it < kBmIts; ++it)
            if (it < its)
                qpre[q_wave + it * kWave + lane] = (uint16_t)(run + inc[it]);
        if (tid == 0)
            a.seg_cnt[cur.sg] = cnt;
        __syncthreads();
        // 3: ranks
        const bool placed = cnt <= places; // the same in every thread
        auto rank_of = [&](uint32_t b) -> uint32_t {
            const uint4 v = quads[b >> 7];
            const uint32_t w = (b >> 5) & 3u, below = (1u << (b & 31u)) - 1u;
            const uint32_t word = w == 0 ? v.x : w == 1 ? v.y : w == 2 ? v.z : v.w;
            const uint32_t r = qpre[b >> 7] + (w > 0 ? __popc(v.x) : 0) + (w > 1 ? __popc(v.y) : 0) + (w > 2 ? __popc(v.z) : 0) +
                               __popc(word & below);
            if (placed)
                place[r] = id0 + b;
            else
                uids[r] = id0 + b;
            return r;
        };
#pragma unroll
        for (int q = 0; q < kBmKeep; ++q)
            if (keep[q] != 0xFFFFFFFFu)
                ranks[q * kBmThreads + tid] = (uint16_t)rank_of(keep[q]);
        for (uint32_t j = kBmKeep * kBmThreads + tid; j < m; j += kBmThreads)
            ranks[j] = (uint16_t)rank_of(ids[j] - id0);
        __syncthreads();
        if (placed)
            for (uint32_t r = tid; r < cnt; r += kBmThreads)
                uids[r] = place[r];
        if (!LISTED)
            return;
        // 4: clear
        if (m * 4u < nq) {
#pragma unroll
            for (int q = 0; q < kBmKeep; ++q)
                if (keep[q] != 0xFFFFFFFFu)
                    words[keep[q] >> 5] = 0u;
            for (uint32_t j = kBmKeep * kBmThreads + tid; j < m; j += kBmThreads)
                words[(ids[j] - id0) >> 5] = 0u;
        } else {
            for (int it = 0; it < its; ++it)
                quads[q_wave + it * kWave + lane] = make_uint4(0, 0, 0, 0);
        }
        __syncthreads();
    }
}

// One workgroup per minibatch: distinct ids before each segment; distinct ids of the minibatch.  The segment
// counters are left all zero for the next hop.  The workgroup that finishes last then turns the minibatches' counts
// into the stacked column offsets (= the next hop's row offsets), the hop's column count, and the next hop's row
// tiles.  When a segment fitted no ranking kernel (flag), the hop's outputs are written as empty: the caller sees the
// flag with the sizes and repeats the call with the per-minibatch kernel on this hop.
// The counts pass from one workgroup to the last one by atomics alone: a fence of every workgroup, which writes its die's whole
// cache back, made two hops of 256 minibatches take 22 us, 16.5 so.
__global__ __launch_bounds__(256) void dd_base_scan_kernel(DedupArgs a, int64_t *mb_coloff, int64_t *ncols_out,
                                                           int64_t *next_tileoff /* k + 2 */, uint32_t *done)
{
    __shared__ uint32_t smem[4];
    __shared__ uint32_t carry_s;
    __shared__ int64_t smem64[4];
    __shared__ int64_t carry64_s, carry64b_s;
    __shared__ uint32_t last_s;
    const bool failed = *a.fallback != 0;
    const int i = blockIdx.x, tid = threadIdx.x;
    if (tid == 0)
        carry_s = 0;
    __syncthreads();
    for (int base = 0; base < a.C; base += 256) {
        const int c = base + tid;
        uint32_t v = 0;
        if (c < a.C) {
            v = a.seg_cnt[(int64_t)i * a.C + c];
            a.seg_cnt[(int64_t)i * a.C + c] = 0;
        }
        uint32_t total;
        const uint32_t ex = block_exclusive_scan<uint32_t, 256>(v, smem, total);
        const uint32_t carry = carry_s;
        if (c < a.C)
            a.bin_base[(int64_t)i * a.stride + c] = carry + ex;
        __syncthreads();
        if (tid == 0)
            carry_s = carry + total;
        __syncthreads();
    }
    if (tid == 0) {
        __hip_atomic_store(&a.mb_count[i], failed ? (int64_t)0 : (int64_t)carry_s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last_s = arrive_last(done, (uint32_t)a.k) ? 1u : 0u;
    }
    __syncthreads();
    if (!last_s)
        return;
    if (tid == 0) {
        carry64_s = 0;
        carry64b_s = 0;
    }
    __syncthreads();
    int64_t most = 0;
    for (int32_t base = 0; base < a.k; base += 256) {
        const int32_t j = base + tid;
        const int64_t v = j < a.k ? __hip_atomic_load(&a.mb_count[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
        const int64_t tiles = (v + kRowTile - 1) / kRowTile;
        most = tiles > most ? tiles : most;
        int64_t total, total_t;
        const int64_t ex = block_exclusive_scan<int64_t, 256>(v, smem64, total);
        const int64_t ex_t = block_exclusive_scan<int64_t, 256>(tiles, smem64, total_t);
        const int64_t carry = carry64_s, carry_t = carry64b_s;
        if (j < a.k) {
            mb_coloff[j] = carry + ex;
            next_tileoff[j] = carry_t + ex_t;
        }
        __syncthreads();
        if (tid == 0) {
            carry64_s = carry + total;
            carry64b_s = carry_t + total_t;
        }
        __syncthreads();
    }
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) {
        const int64_t o = __shfl_xor(most, d, kWave);
        most = o > most ? o : most;
    }
    if ((tid & (kWave - 1)) == 0)
        smem64[tid / kWave] = most;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 4; ++w)
            most = smem64[w] > most ? smem64[w] : most;
        mb_coloff[a.k] = carry64_s;
        *ncols_out = carry64_s;
        next_tileoff[a.k] = carry64b_s;
        next_tileoff[a.k + 1] = most;
    }
}

// The cut in reverse: tile t appended, for every segment c, one run of ids to the segment; the ranks of those
// ids lie at the same places.  Per tile: the runs' ranks are read back in the order of the cut (wide loads; the run of a place
// follows from a bit per place where a run begins), the distinct ids before the segment are added, and every position reads its
// column from the place that the cut left for it.  Memory and the latency of the scattered short runs bound it: all 16 ranks of a
// thread are in flight at once, a run's number and a position's place share a register, so that four workgroups of 64 registers
// share a compute unit.  128 x 586 k ids: 299 us with two workgroups and four loads in flight, 171 with four and a word of 32 bits
// per position that scattered the ranks, 161 with 16 bits and one random access of LDS per entry, 137 since tiles begin at lines.
template <int TILE, int NT, bool PAST>
__global__ __launch_bounds__(NT, 8) void dd_unsplit_kernel(DedupArgs a, const int64_t *__restrict__ tileoff)
{
    // stage[TILE]; a bit per place of the cut's order where a run begins; then, by rank among the tile's runs, 2 C words: start in
    // global - start in the tile, base
    extern __shared__ __attribute__((aligned(16))) uint32_t unsplit_lds[]; // (read by 64 bits as well)
    __shared__ uint32_t smem[NT / kWave];
    __shared__ uint32_t carry_s;
    if (*a.fallback)
        return;
    static_assert(TILE <= 1 << 16 && TILE / kWave == 2 * kWave, "two words of 64 places per lane");
    uint32_t *stage = unsplit_lds, *starts = unsplit_lds + TILE;
    uint32_t *delta = starts + TILE / 32, *base_l = delta + a.C;
    const int64_t ntiles = uniform_load(tileoff + a.k);
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        uint32_t tid = threadIdx.x;
        asm volatile("" : "+v"(tid)); // (places: computed anew for every tile, not kept in registers)
        __builtin_assume(tid < NT);
        const uint32_t lane = tid & (kWave - 1), wave = scalar(tid / kWave);
        const int i = locate_uniform(tileoff, a.k, t);
        const int64_t e0 = uniform_load(a.mb_edgeoff + i);
        const uint32_t N = (uint32_t)(uniform_load(a.mb_edgeoff + i + 1) - e0);
        uint32_t j0, jend;
        cut_tile(e0, N, (uint32_t)(t - uniform_load(tileoff + i)), j0, jend);
        const int n = (int)scalar(jend - j0);
        int left = n - (int)tid;
        const uint16_t *__restrict__ loc = a.loc + scalar(e0 + j0);
        uint32_t place[TILE / NT]; // in the cut's order; later the run that has place q NT + tid, in the upper half
#pragma unroll
        for (int q = 0; q < TILE / NT; ++q)
            place[q] = left > q * NT ? (loc + q * NT)[tid] : 0;
        if (tid == 0)
            carry_s = 0;
        if (tid < TILE / 32)
            starts[tid] = 0;
        __syncthreads();
        const uint32_t *__restrict__ run_gpos = a.run_gpos + t * a.C, *__restrict__ run_cnt = a.run_cnt + t * a.C;
        for (int base = 0; base < a.C; base += NT) {
            const int c = base + (int)tid;
            const uint32_t v = c < a.C ? run_cnt[c] : 0u;
            const uint32_t one = v ? 1u << 16 | v : 0u; // runs and entries (the last run's sum does not count)
            uint32_t total;
            const uint32_t ex = carry_s + block_exclusive_scan<uint32_t, NT>(one, smem, total);
            if (v) {
                const uint32_t rank = ex >> 16, off = ex & 0xFFFFu;
                delta[rank] = run_gpos[c] - off;
                base_l[rank] = a.bin_base[(int64_t)i * a.stride + c];
                atomicOr(&starts[off >> 5], 1u << (off & 31u));
            }
            __syncthreads();
            if (tid == 0)
                carry_s += total;
            __syncthreads();
        }
        // runs that begin before each word of 64 places: every wave for itself, word x in lane x, word x + 64 in its upper half
        const uint64_t *words = reinterpret_cast<const uint64_t *>(starts);
        const uint64_t low = words[lane], high = words[lane + kWave];
        const uint32_t low_c = __popcll(low), high_c = __popcll(high);
        const uint32_t low_upto = wave_inclusive_scan_dpp(low_c);
        const uint32_t high_upto = wave_inclusive_scan_dpp(high_c) + (uint32_t)__builtin_amdgcn_readlane((int)low_upto, kWave - 1);
        const uint16_t *__restrict__ ranks = a.ranks + scalar(e0);
        uint32_t r[TILE / NT];
#pragma unroll
        for (int q = 0; q < TILE / NT; ++q) { // all of a thread's rank loads in flight
            const int word = q * (NT / kWave) + (int)wave;
            const int of = word & (kWave - 1);
            if (q % 4 == 0)
                asm volatile("" : "+v"(tid), "+v"(left) : : "memory"); // (four at a time: all of their places at once do not fit the registers)
            const bool upper = q * (NT / kWave) >= kWave;
            const uint64_t m = (uint64_t)lane_value((int64_t)(upper ? high : low), of);
            const uint32_t before = (uint32_t)__builtin_amdgcn_readlane((int)(upper ? high_upto - high_c : low_upto - low_c), of);
            const uint32_t run = before + (uint32_t)(m & 1u) + bits_below(m >> 1) - 1u;
            r[q] = left > q * NT ? ranks[delta[run] + q * NT + tid] : 0;
            place[q] |= run << 16;
        }
#pragma unroll
        for (int q = 0; q < TILE / NT; ++q)
            if (left > q * NT)
                stage[q * NT + tid] = r[q] + base_l[place[q] >> 16];
        __syncthreads();
        int32_t *__restrict__ col = a.col + scalar(e0 + j0);
#pragma unroll
        for (int q = 0; q < TILE / NT; ++q)
            if (left > q * NT) {
                const int32_t column = (int32_t)stage[place[q] & 0xFFFFu];
                if (PAST) // a.past
                    __builtin_nontemporal_store(column, (col + q * NT) + tid);
                else
                    (col + q * NT)[tid] = column;
            }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------------
// Segments of unequal width.  Ids that crowd parts of [0, n) (ids sorted by degree put every hub at one end)
// overfill segments of equal width.  The hop's staged ids are sampled (every 8th block of 2048) into a histogram
// over cells of 2^fshift ids; the cells are then dealt to segments in id order so that every segment holds about
// the same share of the sample -- a cell that alone holds more stays a segment of its own, narrow enough for the
// bitmap kernel.  The table is the same for all minibatches of the hop (they sample the same graph), and a
// recycled result keeps it for the next call.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void dd_hist_kernel(const int32_t *__restrict__ col, const int64_t *__restrict__ nnz_ptr,
                                                      int32_t fshift, int32_t cells, uint32_t *__restrict__ hist)
{
    __shared__ uint32_t h[kMaxCells + 1];
    const int tid = threadIdx.x;
    for (int x = tid; x <= cells; x += 256)
        h[x] = 0;
    __syncthreads();
    const int64_t nnz = *nnz_ptr;
    for (int64_t b0 = (int64_t)blockIdx.x * 8 * 2048; b0 < nnz; b0 += (int64_t)gridDim.x * 8 * 2048) {
        uint32_t g[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t j = b0 + q * 256 + tid;
            g[q] = j < nnz ? (uint32_t)col[j] : 0xFFFFFFFFu;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (g[q] != 0xFFFFFFFFu)
                atomicAdd(&h[g[q] >> fshift], 1u);
    }
    __syncthreads();
    for (int x = tid; x < cells; x += 256)
        if (h[x])
            atomicAdd(&hist[x], h[x]);
}

// one workgroup: thread t owns cells 4 t .. 4 t + 3
__global__ __launch_bounds__(1024) void dd_table_kernel(const uint32_t *__restrict__ hist, const int64_t *__restrict__ nnz_ptr,
                                                        int32_t k, int32_t cells, int32_t C, int32_t target_per_mb,
                                                        int32_t max_cells, uint16_t *__restrict__ tab,
                                                        uint32_t *__restrict__ seg_first)
{
    __shared__ uint64_t smem[16];
    __shared__ uint32_t smem32[16];
    const int tid = threadIdx.x;
    uint64_t h[4], mine = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int cell = 4 * tid + u;
        h[u] = cell < cells ? hist[cell] : 0u;
        mine += h[u];
    }
    uint64_t S;
    uint64_t before = block_exclusive_scan<uint64_t, 1024>(mine, smem, S);
    // ids of the sample per segment: the share target_per_mb has in a minibatch's ids, and never so few that more
    // than C segments come out (breaks forced by the width limit counted in)
    const uint64_t per_mb = (uint64_t)(*nnz_ptr / k) + 1u;
    const int64_t forced = cells / max_cells + 2;
    const uint64_t room = (uint64_t)(C - forced > 1 ? C - forced : 1);
    uint64_t target = S * (uint64_t)target_per_mb / per_mb + 1u;
    if (target < S / room + 1u)
        target = S / room + 1u;
    uint32_t flags = 0, nflag = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int cell = 4 * tid + u;
        if (cell < cells) {
            const uint64_t prev_before = cell ? before - (u ? h[u - 1] : (uint64_t)hist[cell - 1]) : 0u;
            const bool brk = cell == 0 || before / target != prev_before / target || cell / max_cells != (cell - 1) / max_cells;
            flags |= brk ? 1u << u : 0u;
            nflag += brk ? 1u : 0u;
        }
        before += h[u];
    }
    uint32_t nseg;
    uint32_t seg = block_exclusive_scan<uint32_t, 1024>(nflag, smem32, nseg); // segments that start before this thread's cells
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int cell = 4 * tid + u;
        if (cell < cells) {
            if (flags & (1u << u)) {
                seg_first[seg] = (uint32_t)cell;
                ++seg;
            }
            tab[cell] = (uint16_t)(seg - 1u);
        }
    }
    if (tid == 0)
        tab[cells] = (uint16_t)(nseg - 1u); // ids at the very end of the last cell's range never occur; kept in bounds
    for (uint32_t c = nseg + tid; c <= (uint32_t)C; c += 1024)
        seg_first[c] = (uint32_t)cells; // the segments past the last one in use are empty
}

void launch_nw_dedup_table(const Launch &L, const int32_t *col, const int64_t *nnz, int64_t nnz_bound, int64_t n, int32_t k,
                           int32_t fshift, int32_t C, int32_t target_per_mb, int32_t max_wbits, uint32_t *hist,
                           uint16_t *tab, uint32_t *seg_first)
{
    const int32_t cells = (int32_t)(((n > 0 ? n : 1) + (1LL << fshift) - 1) >> fshift); // <= kMaxCells
    int64_t max_cells = max_wbits >= 31 ? (int64_t)cells + 1 : (1LL << (max_wbits > fshift ? max_wbits - fshift : 0));
    if (max_cells > cells)
        max_cells = cells + 1;
    (void)hipMemsetAsync(hist, 0, ((size_t)cells + 1) * sizeof(uint32_t), L.stream);
    hipLaunchKernelGGL(dd_hist_kernel, dim3(grid_for(L, nnz_bound / (8 * 2048) + 1, 2)), dim3(256), 0, L.stream, col, nnz,
                       fshift, cells, hist);
    hipLaunchKernelGGL(dd_table_kernel, dim3(1), dim3(1024), 0, L.stream, hist, nnz, k, cells, C, target_per_mb,
                       (int32_t)max_cells, tab, seg_first);
}

// Workgroups for the tiles of the cut: one each of as many as there are likely to be.  (Of a call that reads no sizes back nnz is a
// bound, several times what there is; a workgroup without a tile takes its time as well.)
static int cut_grid(const Launch &L, const DedupArgs &a, int64_t nnz)
{
    return grid_for(L, cut_tiles_bound(std::min(nnz, a.nnz_tune + a.nnz_tune / 8), a.k), kOnePass);
}

void launch_nw_extract_segments(const Launch &L, const DedupArgs &a, const int64_t *out_rowptr, const int64_t *mb_rowoff,
                                int64_t *mb_coloff, int32_t *col_vertex, int64_t *ncols_out, int64_t *next_tileoff,
                                uint32_t *done, int64_t nnz, bool counted, const StageMark &mark)
{
    mark("dd_plan");
    const int64_t tiles = cut_tiles_bound(nnz, a.k);
    hipLaunchKernelGGL(dd_plan_kernel, dim3(a.k + 1), dim3(256), 0, L.stream, a, out_rowptr, mb_rowoff, counted ? 1 : 0);
    if (!counted) {
        hipLaunchKernelGGL((dd_count_kernel<kCutTile, 512>), dim3(grid_for(L, tiles, 4)), dim3(512), 0, L.stream, a,
                           a.big_tileoff);
        hipLaunchKernelGGL(dd_seg_scan_kernel, dim3(a.k), dim3(256), 0, L.stream, a);
    }
    mark("dd_split");
    { // 8192 ids per step, workgroups of 8 waves, several per compute unit
        void (*const kernels[2])(DedupArgs, const int64_t *) = {dd_split_kernel<kCutTile, kSplitThreads, false>, dd_split_kernel<kCutTile, kSplitThreads, true>};
        static bool attr_set = false;
        const size_t table = ((size_t)kMaxCells + 2) * sizeof(uint16_t);
        if (!attr_set) {
            for (auto *kernel : kernels)
                if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                        (int)(kCutTile * sizeof(uint32_t) + 3 * kMaxSegments * sizeof(uint32_t) + table)) != hipSuccess)
                    (void)hipGetLastError(); // not required on every runtime; a refused launch shows in the caller's error check
            attr_set = true;
        }
        const size_t lds = (size_t)kCutTile * sizeof(uint32_t) + 3 * (size_t)a.C * sizeof(uint32_t) + (a.tab ? table : 0);
        hipLaunchKernelGGL(kernels[a.tab ? 1 : 0], dim3(cut_grid(L, a, nnz)), dim3(kSplitThreads), lds, L.stream, a, a.big_tileoff);
    }
    mark("dd_rank");
    static bool big_attr_set = false;
    if (!big_attr_set) {
        int most = 0;
        for (int shift = 0; shift <= kMaxBitmapShift; ++shift)
            most = std::max(most, (int)dd_bitmap_lds_bytes(shift));
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(dd_bitmap_kernel<false>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, most) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void *>(dd_bitmap_kernel<true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, most) != hipSuccess)
            (void)hipGetLastError(); // not required on every runtime; a refused launch shows in the caller's error check
        big_attr_set = true;
    }
    const size_t bm_lds = dd_bitmap_lds_bytes(a.wbits_max <= kMaxBitmapShift ? a.wbits_max : kMaxBitmapShift);
    const int bm_per_cu = (int)std::max<size_t>(1, std::min<size_t>(2, (size_t)(156 * 1024) / bm_lds));
    const uint32_t places = (uint32_t)bm_places(a.wbits_max <= kMaxBitmapShift ? a.wbits_max : kMaxBitmapShift);
    if (a.by_bitmap) {
        hipLaunchKernelGGL(dd_bitmap_kernel<false>, dim3(a.k, a.C), dim3(kBmThreads),
                           bm_lds, L.stream, a, places);
    } else {
        hipLaunchKernelGGL(dd_rank_kernel, dim3(a.k, a.C), dim3(kRankThreads), 0, L.stream, a);
        if (a.tab || a.cshift <= kMaxBitmapShift) // segments the counting kernel did not take (none can be listed otherwise)
            hipLaunchKernelGGL(dd_bitmap_kernel<true>, dim3(grid_for(L, nnz / 1024 + 1, bm_per_cu)), dim3(kBmThreads),
                               bm_lds, L.stream, a, places);
    }
    hipLaunchKernelGGL(dd_base_scan_kernel, dim3(a.k), dim3(256), 0, L.stream, a, mb_coloff, ncols_out, next_tileoff, done);
    mark("dd_front");
    launch_nw_dedup_front(L, a, mb_coloff, col_vertex, nnz);
    mark("dd_unsplit");
    launch_nw_dedup_unsplit(L, a, nnz);
}

template <bool PAST>
static void launch_unsplit(const Launch &L, const DedupArgs &a, int64_t nnz)
{
    static bool attr_set = false;
    const size_t lds = (size_t)kCutTile * sizeof(uint32_t) + kCutTile / 8 + 2 * (size_t)a.C * sizeof(uint32_t);
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(dd_unsplit_kernel<kCutTile, 512, PAST>),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)(kCutTile * sizeof(uint32_t) + kCutTile / 8 + 2 * kMaxSegments * sizeof(uint32_t))) != hipSuccess)
            (void)hipGetLastError(); // not required on every runtime; a refused launch shows in the caller's error check
        attr_set = true;
    }
    hipLaunchKernelGGL((dd_unsplit_kernel<kCutTile, 512, PAST>), dim3(cut_grid(L, a, nnz)), dim3(512), lds, L.stream, a,
                       a.big_tileoff);
}

void launch_nw_dedup_unsplit(const Launch &L, const DedupArgs &a, int64_t nnz)
{
    if (a.past)
        launch_unsplit<true>(L, a, nnz);
    else
        launch_unsplit<false>(L, a, nnz);
}

} // namespace bms
