// Node-wise hops small enough for one workgroup per minibatch, Sec. 4.1 of arxiv 2311.02909: a whole hop -- P = Q A,
// SAMPLE, EXTRACT -- and every following hop that still fits, in one launch for all minibatches.
//
// What bounds these hops is not memory but the chain: the chip-wide path takes 6 to 10 launches per hop, each of which costs its
// launch (2.4 us of host time, about 4 us of device time) however little it moves.  Here a minibatch's sampled ids never leave
// LDS:
//   seeds    checked against an LDS hash table (range, repeats), copied to the first frontier
//   sample   one row per lane: extent, draws, the chosen neighbours fetched into registers, all at once
//   rank     the entries' places by id: through 16384 buckets of about one id each, or, when the ids crowd some of them, by
//            a sort in counting passes of 8 bits, as many as n has; distinct ids counted: local column of every entry
//            and, in LDS, the distinct ids ascending, which are the next hop's rows
//   place    where the minibatch's rows, entries and columns lie in the stacked arrays follows from the sizes of the
//            minibatches before it.  Every workgroup publishes its hop's sizes in one word and adds up the words before
//            its own.  A workgroup takes its minibatch off a counter when it starts, so the ones it waits for have
//            started earlier and wait for nobody after them: every wait ends, whatever else runs on the chip.
// Measured on 2.4 M vertices, one hop per call, s = 16, whole calls: k minibatches of b seeds here and by the chip-wide path
//   k     b = 64     b = 256    b = 512    b = 1000 (11 k entries per minibatch)
//   1     22, 32     23, 37     27, 39     32, 39 us
//   4     22, 38     24, 48     26, 49     35, 52
//   16    23, 62     24, 69     27, 76     35, 70
//   64    24, 63     26, 71     28, 80     38, 76
//   256   33, 66     36, 78     42, 93     56, 99
// so it takes every hop that fits its LDS (kSmallCap), whatever the number of minibatches; two hops (5, 5) of 4 x 64: 28, 62 us.
#include "bms_device.h"
#include "bms_internal.h"
#include "nw_draws.h"

#include <type_traits>

namespace bms {

constexpr int kSmThreads = 1024;
constexpr int kSmWaves = kSmThreads / kWave;
constexpr int kSmBins = 256;                   // a counting pass takes 8 bits
constexpr int kSmBuckets = kSmallBuckets;
constexpr int kSmCrowd = 64;                   // ids per bucket, at most
constexpr int kSmRounds = kSmallCap / kSmThreads; // entries per thread, at most: entry e is thread e mod 1024's
constexpr int kSmMaskWords = kSmallCap / 32;
// words: bucket counters and starts, or the counters of the passes; one bit per place, set bits before each word
constexpr int kSmSort = kSmBuckets / 4 + kSmBuckets / 8, kSmWork = kSmSort + 2 * kSmMaskWords;
constexpr uint32_t kSmEmpty = 0xFFFFFFFFu;
static_assert(kSmSort >= kSmWaves * kSmBins && kSmSort >= 2 * kSmallCap / kWave && kSmBuckets == 16 * kSmThreads &&
              kSmMaskWords <= kSmThreads && kSmallCap <= 16384, "work area out of step");

__device__ __forceinline__ int64x2_a8 small_extent(const NwSmall &a, int32_t v)
{
    int64x2_a8 extent = {0, 0};
    if (v >= 0 && (int64_t)v < a.n) // a seed outside [0, n) is reported by the seed check: never read out of bounds
        extent = row_extent(a.A_rowptr, v);
    return extent;
}

// The R rows of a hop, one per lane: front[r], the row's vertex, becomes its offset in the minibatch's entries; chosen neighbours,
// or their places in A_col (flat), go to key[R + offset ..].  v, extent: of row threadIdx.x (v < 0: there is none).
template <int S, bool REPLACE>
__device__ __forceinline__ int32_t small_sample_rows(const NwSmall &a, uint64_t hopkey, int32_t s, uint32_t mb, int32_t R, int32_t v,
                                                     int64x2_a8 extent, uint32_t *front, uint32_t *key, uint32_t *wsum)
{
    const int tid = threadIdx.x;
    int32_t run = 0;
    for (int32_t r0 = 0; r0 < R; r0 += kSmThreads) {
        const int32_t r = r0 + tid, now = v;
        const int64_t beg = extent[0];
        const int32_t deg = (int32_t)(extent[1] - extent[0]);
        if (r0 + kSmThreads < R) {
            v = r + kSmThreads < R ? (int32_t)front[r + kSmThreads] : -1;
            extent = small_extent(a, v);
        }
        int32_t cnt = deg < s ? deg : s;
        uint32_t c[S];
        if (REPLACE && deg > 0)
            cnt = replace_draws<S>(row_key(hopkey, mb, (uint32_t)now), (uint32_t)deg, s, c);
        uint32_t total;
        const int32_t loc = run + (int32_t)block_exclusive_scan<uint32_t, kSmThreads>((uint32_t)cnt, wsum, total);
        if (r < R) {
            front[r] = (uint32_t)loc;
            if (a.self_entry)
                key[r] = (now >= 0 && (int64_t)now < a.n) ? (uint32_t)now : 0u;
        }
        if (cnt > 0) {
            uint32_t *dst = key + (a.self_entry ? R : 0) + loc;
            if (!REPLACE && deg > s)
                distinct_draws<S>(row_key(hopkey, mb, (uint32_t)now), (uint32_t)deg, s, c);
            if (a.flat) { // the neighbours follow when all rows have chosen theirs
                int32_t m = 0;
#pragma unroll
                for (int j = 0; j < S; ++j)
                    if (REPLACE ? (j < s && (j == 0 || c[j] != c[j - 1])) : j < cnt)
                        dst[m++] = (uint32_t)beg + (!REPLACE && deg <= s ? (uint32_t)j : c[j]);
            } else {
                const int32_t *__restrict__ src = a.A_col + beg;
                int32_t m = 0;
#pragma unroll
                for (int j = 0; j < S; ++j) {
                    if (REPLACE ? (j < s && (j == 0 || c[j] != c[j - 1])) : j < cnt)
                        dst[m++] = (uint32_t)src[!REPLACE && deg <= s ? (uint32_t)j : c[j]];
                    __builtin_amdgcn_sched_barrier(0); // addresses one at a time: they do not all fit the registers
                }
            }
        }
        run += (int32_t)total;
    }
    return run;
}

// Local columns of N entries, id[] (entry u * 1024 + threadIdx.x in id[u]), by 16384 buckets of equal id ranges (about one id each
// when n is large): counted (8 bits per bucket), scanned, every id to its bucket's places, and there compared with the few
// others: an entry's first possible place, bucket's start + smaller ids in it, gets a bit, and its column is the number of
// bits before.  Returns false, with key[] as it was, when a bucket holds more than kSmCrowd ids (a hub that many rows
// sampled, ids crowded into a narrow range): the counting passes take those.  key: cap words that may be overwritten; the counters
// and the bits are zero on entry.
template <int ROUNDS>
__device__ __forceinline__ bool small_rank_buckets(const NwSmall &a, const uint32_t (&id)[ROUNDS], uint32_t (&col)[ROUNDS],
                                                   uint32_t *key, uint32_t *work, int32_t N, uint32_t *wsum, uint32_t *crowded_s,
                                                   uint32_t &distinct)
{
    const int tid = threadIdx.x;
    uint32_t *cnt = work;                                               // 4 counters of 8 bits per word
    uint16_t *start = reinterpret_cast<uint16_t *>(work + kSmBuckets / 4); // ids before the word's first bucket
    uint32_t *mask = work + kSmSort, *before = mask + kSmMaskWords;
    auto bucket = [&](uint32_t x) { return a.bucket_mul ? __umulhi(x, a.bucket_mul) : x; };
    const int32_t mine = N - tid; // entries from the thread's first on
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u)
        if (u * kSmThreads < mine) {
            const uint32_t d = bucket(id[u]);
            col[u] = atomicAdd(&cnt[d >> 2], 1u << (8u * (d & 3u)));
        }
    bool crowded = false; // seen by whoever adds the first id too many, whatever the counter does after that
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u)
        if (u * kSmThreads < mine) {
            col[u] = (col[u] >> (8u * (bucket(id[u]) & 3u))) & 255u;
            crowded |= col[u] >= (uint32_t)kSmCrowd;
        }
    if (crowded)
        *crowded_s = 1;
    __syncthreads();
    if (*crowded_s)
        return false; // the same for the whole workgroup
    {
        const uint4 w = reinterpret_cast<const uint4 *>(cnt)[tid]; // kSmBuckets / 4 = 4 words per thread
        const uint32_t x[4] = {w.x, w.y, w.z, w.w};
        uint32_t c[4], sum = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            c[u] = (x[u] & 255u) + ((x[u] >> 8) & 255u) + ((x[u] >> 16) & 255u) + (x[u] >> 24);
            sum += c[u];
        }
        uint32_t total;
        uint32_t ex = block_exclusive_scan<uint32_t, kSmThreads>(sum, wsum, total);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            start[4 * tid + u] = (uint16_t)ex;
            ex += c[u];
        }
    }
    __syncthreads();
    // col[u]: first place (14 bits) and size of the entry's bucket
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u)
        if (u * kSmThreads < mine) {
            const uint32_t d = bucket(id[u]), w = cnt[d >> 2], sh = 8u * (d & 3u);
            const uint32_t lower = w & ((1u << sh) - 1u); // counters of the word's buckets before d: at most three of them
            const uint32_t s0 = (uint32_t)start[d >> 2] + (lower & 255u) + ((lower >> 8) & 255u) + ((lower >> 16) & 255u);
            key[s0 + col[u]] = id[u];
            col[u] = s0 | ((w >> sh) & 255u) << 14;
        }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u)
        if (u * kSmThreads < mine) {
            const uint32_t s0 = col[u] & 16383u, n = col[u] >> 14;
            uint32_t to = s0;
            if (n > 1u) {
                const uint32_t x0 = key[s0], x1 = key[s0 + 1], x2 = key[s0 + min(2u, n - 1u)], x3 = key[s0 + min(3u, n - 1u)];
                to += (x0 < id[u] ? 1u : 0u) + (x1 < id[u] ? 1u : 0u) + (n > 2u && x2 < id[u] ? 1u : 0u) +
                      (n > 3u && x3 < id[u] ? 1u : 0u);
                for (uint32_t q = 4; q < n; ++q)
                    to += key[s0 + q] < id[u] ? 1u : 0u;
            }
            atomicOr(&mask[to >> 5], 1u << (to & 31u));
            col[u] = to;
        }
    __syncthreads();
    const uint32_t bits = tid < kSmMaskWords ? (uint32_t)__popc(mask[tid < kSmMaskWords ? tid : 0]) : 0u;
    const uint32_t ex = block_exclusive_scan<uint32_t, kSmThreads>(bits, wsum, distinct);
    if (tid < kSmMaskWords)
        before[tid] = ex;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u)
        if (u * kSmThreads < mine)
            col[u] = before[col[u] >> 5] + (uint32_t)__popc(mask[col[u] >> 5] & ((1u << (col[u] & 31u)) - 1u));
    return true;
}

// Sorted order of N ids by stable counting passes of 8 bits, whatever the ids: the permutation moves from one array to the other.
__device__ __forceinline__ uint16_t *small_sort_radix(int32_t idbits, const uint32_t *key, uint16_t *from, uint16_t *to,
                                                      uint32_t *hist, int32_t N, int32_t e0, int32_t e1, int wave, uint32_t *wsum)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const uint64_t below = (1ull << lane) - 1ull;
    for (int32_t e = e0 + lane; e < e1; e += kWave)
        from[e] = (uint16_t)e;
    uint32_t *mine = hist + wave * kSmBins;
    for (int32_t shift = 0; shift < idbits; shift += 8) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kSmBins / kWave; ++q)
            mine[q * kWave + lane] = 0;
        __builtin_amdgcn_wave_barrier();
        for (int32_t e = e0 + lane; e < e1; e += kWave)
            atomicAdd(&mine[(key[from[e]] >> shift) & (kSmBins - 1)], 1u);
        __syncthreads();
        { // exclusive scan in (digit, wave) order: thread t takes waves 4 (t & 3) .. + 3 of digit t / 4
            uint32_t x[4];
            const int d = tid >> 2, w0 = (tid & 3) * 4;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                x[u] = hist[(w0 + u) * kSmBins + d];
            uint32_t total;
            uint32_t ex = block_exclusive_scan<uint32_t, kSmThreads>(x[0] + x[1] + x[2] + x[3], wsum, total);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                hist[(w0 + u) * kSmBins + d] = ex;
                ex += x[u];
            }
        }
        __syncthreads();
        for (int32_t eb = e0; eb < e1; eb += kWave) {
            const bool valid = eb + lane < e1;
            const uint32_t p = valid ? (uint32_t)from[eb + lane] : 0u;
            const uint32_t d = valid ? (key[p] >> shift) & (kSmBins - 1) : 0u;
            uint64_t peers = __ballot(valid); // lanes with the same digit
#pragma unroll
            for (int bit = 0; bit < 8; ++bit) {
                const uint64_t set = __ballot((d >> bit) & 1u);
                peers &= ((d >> bit) & 1u) ? set : ~set;
            }
            const uint32_t rank = (uint32_t)__popcll(peers & below);
            const uint32_t base = mine[d];
            __builtin_amdgcn_wave_barrier();
            if (valid && rank == 0)
                mine[d] = base + (uint32_t)__popcll(peers);
            __builtin_amdgcn_wave_barrier();
            if (valid)
                to[base + rank] = (uint16_t)p;
        }
        uint16_t *t = from;
        from = to;
        to = t;
    }
    __syncthreads();
    return from;
}

// The same by the sorted order: heads of its runs of equal ids, counted.  pos: 2 cap words of 16 bits; key[]: the ids.
template <int ROUNDS>
__device__ __forceinline__ void small_rank_radix(const NwSmall &a, uint32_t (&col)[ROUNDS], const uint32_t *key, uint16_t *pos,
                                                 uint32_t *work, int32_t N, uint32_t *wsum, uint32_t &distinct)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave); // the same in every lane: loop bounds stay scalar
    const uint64_t below = (1ull << lane) - 1ull;
    // every wave owns `per` consecutive places, 64 of them in each of its steps
    const int32_t per = ((N + kSmWaves - 1) / kSmWaves + kWave - 1) / kWave * kWave;
    const int32_t e0 = wave * per, e1 = min(e0 + per, N);
    uint16_t *by = small_sort_radix(a.idbits, key, pos, pos + a.cap, work, N, e0, e1, wave, wsum);
    uint16_t *rank_of = by == pos ? pos + a.cap : pos; // the other array is free
    unsigned long long *mask = reinterpret_cast<unsigned long long *>(work); // one mask per step
    uint32_t heads = 0;                                                      // of this wave's part
    for (int32_t eb = e0; eb < e1; eb += kWave) {
        const int32_t e = eb + lane;
        const uint32_t id = e < e1 ? key[by[e]] : 0u;
        uint32_t prev = __shfl_up(id, 1, kWave);
        if (lane == 0 && e > 0)
            prev = key[by[e - 1]];
        const uint64_t hm = __ballot(e < e1 && (e == 0 || prev != id));
        if (lane == 0)
            mask[eb / kWave] = hm;
        heads += (uint32_t)__popcll(hm);
    }
    if (lane == 0)
        wsum[wave] = heads;
    __syncthreads();
    uint32_t run = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kSmWaves; ++w) {
        run += w < wave ? wsum[w] : 0u;
        all += wsum[w];
    }
    distinct = all;
    const int32_t mine = N - tid;
    for (int32_t eb = e0; eb < e1; eb += kWave) {
        const uint64_t hm = mask[eb / kWave];
        if (eb + lane < e1)
            rank_of[by[eb + lane]] = (uint16_t)(run + (uint32_t)__popcll(hm & (below | (1ull << lane))) - 1u);
        run += (uint32_t)__popcll(hm);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u)
        if (u * kSmThreads < mine)
            col[u] = rank_of[u * kSmThreads + tid];
}

// Sums over the workgroup of three values per thread (a wave's fit 32 bits); `room`: 3 * kSmWaves words
__device__ __forceinline__ void small_sums(uint32_t x, uint32_t y, uint32_t z, uint32_t *room, int64_t &sx, int64_t &sy, int64_t &sz)
{
    const int wave = threadIdx.x / kWave;
    x = wave_inclusive_scan_dpp(x);
    y = wave_inclusive_scan_dpp(y);
    z = wave_inclusive_scan_dpp(z);
    if ((threadIdx.x & (kWave - 1)) == kWave - 1) {
        room[wave] = x;
        room[kSmWaves + wave] = y;
        room[2 * kSmWaves + wave] = z;
    }
    __syncthreads();
    sx = sy = sz = 0;
#pragma unroll
    for (int w = 0; w < kSmWaves; ++w) {
        sx += room[w];
        sy += room[kSmWaves + w];
        sz += room[2 * kSmWaves + w];
    }
}

// One compute unit, a chain of trips to memory and barriers, and for thousands of entries LDS.  Entries stay in
// registers from the gather to the output, so that an entry's column costs about a dozen LDS accesses and no indirect ones (each
// id was looked up through a permutation in LDS before); the extract exists for 1, 4 and 16 entries per thread, as the code of
// rounds that a hop does not have costs too: about 0.5 us in each of 8 phases, fetching instructions only to jump over them.
// First hop of 1024 seeds, fanout 15, 11 k entries: 43 -> 33 us (gather 7 -> 2, extract 20 -> 11, output 5 -> 2.5); two hops (5, 5)
// of 4 x 64: 27.5 -> 22.3 us.
// SMAX: the largest fanout of the hops, 16 or 32 (the position lists of 32 draws spill; 16 do not)
template <bool REPLACE, int SMAX>
__global__ __launch_bounds__(kSmThreads) void nw_small_kernel(NwSmall a)
{
    extern __shared__ uint32_t small_lds[]; // key[cap], front[cap] (which change places from hop to hop), work[kSmWork]
    __shared__ uint32_t wsum[kSmWaves], sums_s[3 * kSmWaves];
    __shared__ uint32_t take_s, crowded_s;
    uint32_t *key = small_lds, *front = small_lds + a.cap, *work = small_lds + 2 * a.cap;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    if (tid == 0)
        take_s = atomicAdd(a.ticket, 1u) - a.ticket0;
    auto clear = [&] { // bucket counters and place bits
        reinterpret_cast<uint4 *>(work)[tid] = make_uint4(0, 0, 0, 0); // kSmBuckets / 4 = 4 words per thread
        if (tid < kSmMaskWords)
            work[kSmSort + tid] = 0;
        if (tid == 0)
            crowded_s = 0;
    };
    clear();
    const int32_t slots = a.seed_slots; // power of two >= 2 b, within key[]
    for (int32_t x = tid; x < slots; x += kSmThreads)
        key[x] = kSmEmpty;
    __syncthreads();
    const int32_t i = __builtin_amdgcn_readfirstlane((int)take_s);
    const bool last = i == a.k - 1;
    if (last) { // scalars that the kernels of the hops that follow on the chip-wide path expect at zero
        if (tid >= a.nhops && tid < a.L)
            a.slots[4 * tid + 2] = 0;
        if (tid == 63)
            a.slots[63] = 0;
    }

    // seeds; the extents of the first of them are fetched meanwhile
    int32_t R = a.b;
    int64_t row0 = (int64_t)i * a.b; // first stacked row
    int32_t v = tid < R ? a.batches[row0 + tid] : -1;
    int64x2_a8 extent = small_extent(a, v);
    if (tid == 0)
        a.mb_rowoff0[i] = row0;
    if (last && tid == 0)
        a.mb_rowoff0[a.k] = row0 + a.b;
    for (int32_t j = tid; j < a.b; j += kSmThreads) {
        const int32_t x = j == tid ? v : a.batches[row0 + j];
        front[j] = (uint32_t)x;
        a.row_vertex0[row0 + j] = x;
        if (x < 0 || (int64_t)x >= a.n) {
            a.seed_flags[0] = 1;
            continue;
        }
        uint32_t slot = ((uint32_t)x * 0x9E3779B1u) >> a.seed_shift;
        while (true) {
            const uint32_t old = atomicCAS(&key[slot], kSmEmpty, (uint32_t)x);
            if (old == kSmEmpty)
                break;
            if (old == (uint32_t)x) {
                a.seed_flags[1] = 1;
                break;
            }
            slot = (slot + 1u) & (uint32_t)(slots - 1);
        }
    }
    __syncthreads();

    int64_t rows_total = (int64_t)a.k * a.b; // (of the last minibatch only)
    for (int32_t h = 0; h < a.nhops; ++h) {
        const NwSmallHop &H = a.hop[h];
        const uint32_t mb = a.mb_base + (uint32_t)i;
        int32_t nnz;
        if (H.s <= 4)
            nnz = small_sample_rows<4, REPLACE>(a, H.hopkey, H.s, mb, R, v, extent, front, key, wsum);
        else if (H.s <= 8)
            nnz = small_sample_rows<8, REPLACE>(a, H.hopkey, H.s, mb, R, v, extent, front, key, wsum);
        else if (SMAX == 16 || H.s <= 16)
            nnz = small_sample_rows<16, REPLACE>(a, H.hopkey, H.s, mb, R, v, extent, front, key, wsum);
        else
            nnz = small_sample_rows<SMAX, REPLACE>(a, H.hopkey, H.s, mb, R, v, extent, front, key, wsum);
        const int32_t self = a.self_entry ? R : 0; // entries [0, self): the rows' own vertices, then the sampled ones
        const int32_t N = __builtin_amdgcn_readfirstlane(nnz + self); // the same in all lanes
        __syncthreads();

        uint32_t U; // distinct ids = columns
        const bool tiles_wanted = h == a.nhops - 1 && a.next_tileoff; // of the hop that follows on the chip-wide path
        int64_t edge0 = 0, col0 = 0, tile0 = 0; // entries, columns and row tiles of the minibatches before this one
        int32_t most = 0;
        // EXTRACT of N <= ROUNDS * 1024 entries.  By buckets, or, with the ids in key[], by the sort.  False: the ids crowd some
        // buckets; they are in key[] and nothing else has been done.
        auto extract = [&](auto rounds, auto sorted) __attribute__((always_inline))
        {
            constexpr int ROUNDS = decltype(rounds)::value;
            constexpr bool SORTED = decltype(sorted)::value;
            // the entries' ids, in registers from here on: places in A_col -> the neighbours there, the picks of a row in
            // neighbouring lanes (one request per line), all of them on their way at once
            uint32_t id[ROUNDS], col[ROUNDS];
            const int32_t mine = N - tid, sampled = self - tid; // the thread has entry u when u * 1024 < mine, a sampled one from `sampled` on
#pragma unroll
            for (int u = 0; u < ROUNDS; ++u)
                id[u] = u * kSmThreads < mine ? key[u * kSmThreads + tid] : 0u;
            if (!SORTED && a.flat && nnz > 0) {
#pragma unroll
                for (int u = 0; u < ROUNDS; ++u)
                    if (u * kSmThreads < N) // self entries read place 0
                        col[u] = (uint32_t)a.A_col[u * kSmThreads >= sampled && u * kSmThreads < mine ? id[u] : 0u];
#pragma unroll
                for (int u = 0; u < ROUNDS; ++u)
                    if (u * kSmThreads < N)
                        id[u] = u * kSmThreads >= sampled ? col[u] : id[u];
            }
            if constexpr (SORTED) {
                for (int32_t r = tid; r < R; r += kSmThreads) // front[] serves as the order meanwhile
                    H.rowptr[row0 + r] = front[r];
                __syncthreads();
                small_rank_radix<ROUNDS>(a, col, key, reinterpret_cast<uint16_t *>(front), work, N, wsum, U);
                __syncthreads();
                for (int32_t r = tid; r < R; r += kSmThreads)
                    front[r] = (uint32_t)H.rowptr[row0 + r]; // written by this thread
            } else if (!small_rank_buckets<ROUNDS>(a, id, col, key, work, N, wsum, &crowded_s, U)) {
#pragma unroll
                for (int u = 0; u < ROUNDS; ++u)
                    if (u * kSmThreads < mine)
                        key[u * kSmThreads + tid] = id[u];
                __syncthreads();
                return false;
            }
            // sizes of this minibatch for everyone after it
            unsigned long long *status = a.status + (int64_t)h * a.k;
            if (tid == 0)
                __hip_atomic_store(status + i, ((unsigned long long)a.epoch << 32) | ((unsigned long long)(uint32_t)nnz << 16) | U,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // the distinct ids in order, which are the next hop's rows (equal entries write the same)
#pragma unroll
            for (int u = 0; u < ROUNDS; ++u)
                if (u * kSmThreads < mine)
                    key[col[u]] = id[u];
            most = (int32_t)((U + kRowTile - 1) / kRowTile);
            if (i > 0) {
                uint32_t sum_e = 0, sum_c = 0, sum_t = 0;
                for (int32_t j = tid; j < i; j += kSmThreads) {
                    unsigned long long w;
                    while ((uint32_t)((w = __hip_atomic_load(status + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> 32) != a.epoch)
                        __builtin_amdgcn_s_sleep(2);
                    const int32_t cols = (int32_t)(w & 0xFFFFu), tiles = (cols + kRowTile - 1) / kRowTile;
                    sum_e += (uint32_t)((w >> 16) & 0xFFFFu);
                    sum_c += (uint32_t)cols;
                    sum_t += (uint32_t)tiles;
                    most = tiles > most ? tiles : most;
                }
                small_sums(sum_e, sum_c, sum_t, sums_s, edge0, col0, tile0);
            } else {
                __syncthreads(); // key[] is whole
            }
            if (h + 1 < a.nhops) { // extents of the next hop's first rows
                v = tid < (int32_t)U ? (int32_t)key[tid] : -1;
                extent = small_extent(a, v);
            }
            int64_t *rowptr = H.rowptr + row0;
            for (int32_t r = tid; r < R; r += kSmThreads)
                rowptr[r] = edge0 + front[r];
#pragma unroll
            for (int u = 0; u < ROUNDS; ++u) {
                if (u * kSmThreads < sampled)
                    (H.row_self + row0 + u * kSmThreads)[tid] = (int32_t)col[u];
                else if (u * kSmThreads < mine)
                    (H.col + edge0 - self + u * kSmThreads)[tid] = (int32_t)col[u];
            }
            for (int32_t r = tid; r < (int32_t)U; r += kSmThreads)
                H.col_vertex[col0 + r] = (int32_t)key[r];
            return true;
        };
        using std::integral_constant;
        bool done;
        if (N <= kSmThreads)
            done = extract(integral_constant<int, 1>{}, std::false_type{});
        else if (N <= 4 * kSmThreads)
            done = extract(integral_constant<int, 4>{}, std::false_type{});
        else
            done = extract(integral_constant<int, kSmRounds>{}, std::false_type{});
        if (!done)
            extract(integral_constant<int, kSmRounds>{}, std::true_type{});
        if (tid == 0) {
            H.mb_coloff[i] = col0;
            if (a.host_off) {
                int64_t *to = a.host_off + (int64_t)h * 3 * (a.k + 1) + i;
                to[0] = row0;
                to[a.k + 1] = edge0;
                to[2 * (a.k + 1)] = col0;
                if (last) {
                    to[1] = rows_total;
                    to[a.k + 2] = edge0 + nnz;
                    to[2 * (a.k + 1) + 1] = col0 + U;
                }
            }
        }
        if (tiles_wanted) {
            if (tid == 0)
                a.next_tileoff[i] = tile0;
            if (last) {
#pragma unroll
                for (int d = kWave / 2; d > 0; d >>= 1)
                    most = max(most, __shfl_xor(most, d, kWave));
                if (lane == 0)
                    wsum[wave] = (uint32_t)most;
                __syncthreads();
                if (tid == 0) {
                    for (int w = 0; w < kSmWaves; ++w)
                        most = max(most, (int32_t)wsum[w]);
                    a.next_tileoff[a.k] = tile0 + (U + kRowTile - 1) / kRowTile;
                    a.next_tileoff[a.k + 1] = most;
                }
            }
        }
        if (last) {
            if (tid == 0) {
                H.mb_coloff[a.k] = col0 + U;
                H.rowptr[rows_total] = edge0 + nnz;
                for (int64_t *to : {a.slots, a.host_slots})
                    if (to) {
                        to[4 * h] = edge0 + nnz;
                        to[4 * h + 1] = col0 + U;
                        to[4 * h + 2] = 0;
                    }
            }
            rows_total = col0 + U;
        }
        row0 = col0;
        R = (int32_t)U;
        if (h + 1 < a.nhops) {
            clear();
            __syncthreads(); // front[] has been read, the counters are clear
            uint32_t *rows = key;
            key = front;
            front = rows;
        }
    }
    if (a.arrived)
        announce(a.ticket + 1, (uint32_t)a.k, a.arrived, a.arrival);
}

int launch_nw_small(const Launch &L, const NwSmall &a, bool replace)
{
    int32_t smax = 1;
    for (int32_t h = 0; h < a.nhops; ++h)
        smax = a.hop[h].s > smax ? a.hop[h].s : smax;
    void (*const kernels[4])(NwSmall) = {nw_small_kernel<false, 16>, nw_small_kernel<false, 32>, nw_small_kernel<true, 16>,
                                         nw_small_kernel<true, 32>};
    static bool attr_set = false;
    if (!attr_set) {
        for (auto *kernel : kernels)
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)((2 * (size_t)kSmallCap + kSmWork) * sizeof(uint32_t))) != hipSuccess)
                (void)hipGetLastError(); // not required on every runtime; the launch below reports real failures
        attr_set = true;
    }
    const size_t lds = (2 * (size_t)a.cap + kSmWork) * sizeof(uint32_t);
    hipLaunchKernelGGL(kernels[(replace ? 2 : 0) + (smax > 16 ? 1 : 0)], dim3(a.k), dim3(kSmThreads), lds, L.stream, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

} // namespace bms
