// Node-wise hops small enough for one workgroup per minibatch, Sec. 4.1 of arxiv 2311.02909: a whole hop -- P = Q A,
// SAMPLE, EXTRACT -- and every following hop that still fits, in one launch for all minibatches.
//
// What bounds these hops is not memory but the chain: the chip-wide path takes 6 to 10 launches per hop, each of which costs its
// launch (2.4 us of host time, about 4 us of device time) however little it moves.  Here a minibatch's sampled ids never leave
// LDS:
//   seeds    checked against an LDS hash table (range, repeats), copied to the first frontier
//   sample   one row per lane: extent, draws, the chosen neighbours gathered into LDS
//   sort     the positions by id: through 16384 buckets of about one id each, or, when the ids crowd some of them, by
//            counting passes of 8 bits, as many as n has
//   rank     heads of the runs of equal ids, counted: local column of every position, distinct ids ascending
//   place    where the minibatch's rows, entries and columns lie in the stacked arrays follows from the sizes of the
//            minibatches before it.  Every workgroup publishes its hop's sizes in one word and adds up the words before
//            its own.  A workgroup takes its minibatch off a counter when it starts, so the ones it waits for have
//            started earlier and wait for nobody after them: every wait ends, whatever else runs on the chip.
// Measured on 2.4 M vertices, one hop per call, s = 16, whole calls: k minibatches of b seeds here and by the chip-wide path
//   k     b = 64     b = 256    b = 512    b = 1000 (11 k entries per minibatch)
//   1     26, 42     28, 50     34, 50     46, 51 us
//   4     26, 51     28, 61     34, 63     48, 63
//   16    25, 67     29, 81     35, 74     48, 76
//   64    27, 68     31, 84     37, 78     52, 85
//   256   37, 80     45, 96     54, 98     73, 123
// so it takes every hop that fits its LDS (kSmallCap), whatever the number of minibatches; two hops (5, 5) of 4 x 64: 57 us.
#include "bms_device.h"
#include "bms_internal.h"
#include "nw_draws.h"

namespace bms {

constexpr int kSmThreads = 1024;
constexpr int kSmWaves = kSmThreads / kWave;
constexpr int kSmBins = 256;                   // a counting pass takes 8 bits
constexpr int kSmBuckets = kSmallBuckets;
constexpr int kSmCrowd = 64;                   // ids per bucket, at most
constexpr int kSmWork = kSmBuckets / 4 + kSmBuckets / 8; // words: bucket counters and starts, or the counters of the passes
constexpr int kSmGather = 8;                    // reads of A_col in flight per lane
constexpr uint32_t kSmEmpty = 0xFFFFFFFFu;
static_assert(kSmWork >= kSmWaves * kSmBins && kSmWork >= 2 * kSmallCap / kWave && kSmBuckets == 16 * kSmThreads, "work area out of step");

// rows r0 .. r0 + nr - 1 (one per lane) of a hop: local offsets of the rows, chosen neighbours into key[R + offset ..]
template <int S, bool REPLACE>
__device__ __forceinline__ int32_t small_sample_rows(const NwSmall &a, uint64_t hopkey, int32_t s, uint32_t mb,
                                                     const int32_t *__restrict__ rows, int32_t R, int64_t *__restrict__ rowptr,
                                                     uint32_t *key, uint32_t *wsum)
{
    const int tid = threadIdx.x;
    int32_t run = 0;
    for (int32_t r0 = 0; r0 < R; r0 += kSmThreads) {
        const int32_t r = r0 + tid;
        int32_t v = -1, deg = 0, cnt = 0;
        int64_t beg = 0;
        uint32_t c[S];
        if (r < R) {
            v = rows[r];
            if (v >= 0 && (int64_t)v < a.n) { // a seed outside [0, n) is reported by the seed check: never read out of bounds
                beg = a.A_rowptr[v];
                deg = (int32_t)(a.A_rowptr[v + 1] - beg);
            }
            cnt = deg < s ? deg : s;
            if (REPLACE && deg > 0)
                cnt = replace_draws<S>(row_key(hopkey, mb, (uint32_t)v), (uint32_t)deg, s, c);
        }
        uint32_t total;
        const int32_t loc = run + (int32_t)block_exclusive_scan<uint32_t, kSmThreads>((uint32_t)cnt, wsum, total);
        if (r < R) {
            rowptr[r] = loc; // the entries of the minibatches before this one are added when they are known
            if (a.self_entry)
                key[r] = (v >= 0 && (int64_t)v < a.n) ? (uint32_t)v : 0u;
        }
        if (cnt > 0) {
            uint32_t *dst = key + (a.self_entry ? R : 0) + loc;
            if (!REPLACE && deg > s)
                distinct_draws<S>(row_key(hopkey, mb, (uint32_t)v), (uint32_t)deg, s, c);
            if (a.flat) { // the neighbours follow below
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
    if (a.flat) { // places in A_col -> the neighbours there, the picks of a row in neighbouring lanes (one request per line)
        uint32_t *entry = key + (a.self_entry ? R : 0);
        __syncthreads();
        for (int32_t e0 = tid; e0 < run; e0 += kSmGather * kSmThreads) {
            uint32_t g[kSmGather];
#pragma unroll
            for (int u = 0; u < kSmGather; ++u)
                if (e0 + u * kSmThreads < run)
                    g[u] = (uint32_t)a.A_col[entry[e0 + u * kSmThreads]];
#pragma unroll
            for (int u = 0; u < kSmGather; ++u)
                if (e0 + u * kSmThreads < run)
                    entry[e0 + u * kSmThreads] = g[u];
        }
    }
    return run;
}

// Sorted order of N ids by 16384 buckets of equal id ranges (about one id each when n is large): counted (8 bits per
// bucket), scanned, every id to its bucket's places, and there to its final one by comparing it with the few others.
// Returns the array that holds the order, or null when a bucket holds more than kSmCrowd ids (a hub that many rows
// sampled, ids crowded into a narrow range): the counting passes take those.
__device__ __forceinline__ uint16_t *small_sort_buckets(const NwSmall &a, const uint32_t *key, uint16_t *pa, uint16_t *pb,
                                                        uint32_t *work, int32_t N, uint32_t *wsum, uint32_t *crowded_s)
{
    const int tid = threadIdx.x;
    uint32_t *cnt = work;                                               // 4 counters of 8 bits per word
    uint16_t *start = reinterpret_cast<uint16_t *>(work + kSmBuckets / 4); // ids before the word's first bucket
    auto bucket = [&](uint32_t id) { return a.bucket_mul ? __umulhi(id, a.bucket_mul) : id; };
    reinterpret_cast<uint4 *>(cnt)[tid] = make_uint4(0, 0, 0, 0); // kSmBuckets / 4 = 4 words per thread
    if (tid == 0)
        *crowded_s = 0;
    __syncthreads();
    for (int32_t e = tid; e < N; e += kSmThreads) {
        const uint32_t d = bucket(key[e]), sh = 8u * (d & 3u);
        const uint32_t slot = (atomicAdd(&cnt[d >> 2], 1u << sh) >> sh) & 255u;
        if (slot >= (uint32_t)kSmCrowd)
            *crowded_s = 1; // seen by whoever adds the first id too many, before the counter can run over
        pb[e] = (uint16_t)slot;
    }
    __syncthreads();
    if (*crowded_s)
        return nullptr; // the same for the whole workgroup
    {
        const uint4 w = reinterpret_cast<const uint4 *>(cnt)[tid];
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
    // first place and size of bucket d
    auto place = [&](uint32_t d, uint32_t &n) {
        const uint32_t w = cnt[d >> 2], sh = 8u * (d & 3u);
        n = (w >> sh) & 255u;
        const uint32_t lower = w & ((1u << sh) - 1u); // counters of the word's buckets before d: at most three of them
        return (uint32_t)start[d >> 2] + (lower & 255u) + ((lower >> 8) & 255u) + ((lower >> 16) & 255u);
    };
    for (int32_t e = tid; e < N; e += kSmThreads) {
        uint32_t n;
        pa[place(bucket(key[e]), n) + pb[e]] = (uint16_t)e;
    }
    __syncthreads();
    for (int32_t t = tid; t < N; t += kSmThreads) {
        const uint32_t p = pa[t], id = key[p];
        uint32_t n, to = (uint32_t)t;
        const uint32_t s0 = place(bucket(id), n);
        if (n > 1u) {
            to = s0;
            for (uint32_t q = s0; q < s0 + n; ++q) {
                const uint32_t o = key[pa[q]];
                to += (o < id || (o == id && q < (uint32_t)t)) ? 1u : 0u;
            }
        }
        pb[to] = (uint16_t)p;
    }
    __syncthreads();
    return pb;
}

// The same by stable counting passes of 8 bits, whatever the ids: the permutation moves from one array to the other.
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

// SMAX: the largest fanout of the hops, 16 or 32 (the position lists of 32 draws spill; 16 do not)
template <bool REPLACE, int SMAX>
__global__ __launch_bounds__(kSmThreads) void nw_small_kernel(NwSmall a)
{
    extern __shared__ uint32_t small_lds[]; // key[cap], pos[2][cap] (16 bits), work[kSmWork]
    __shared__ uint32_t wsum[kSmWaves];
    __shared__ int64_t wsum64[kSmWaves];
    __shared__ uint32_t take_s, crowded_s;
    uint32_t *key = small_lds;
    uint16_t *pos = reinterpret_cast<uint16_t *>(small_lds + a.cap);
    uint32_t *work = small_lds + 2 * a.cap;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave); // the same in every lane: loop bounds stay scalar
    const uint64_t below = (1ull << lane) - 1ull;
    if (tid == 0)
        take_s = atomicAdd(a.ticket, 1u) - a.ticket0;
    __syncthreads();
    const int32_t i = __builtin_amdgcn_readfirstlane((int)take_s);
    const bool last = i == a.k - 1;
    if (last) { // scalars that the kernels of the hops that follow on the chip-wide path expect at zero
        if (tid >= a.nhops && tid < a.L)
            a.slots[4 * tid + 2] = 0;
        if (tid == 63)
            a.slots[63] = 0;
    }

    // seeds
    int32_t R = a.b;
    int64_t row0 = (int64_t)i * a.b; // first stacked row
    {
        const int32_t slots = a.seed_slots; // power of two >= 2 b, within key[]
        for (int32_t x = tid; x < slots; x += kSmThreads)
            key[x] = kSmEmpty;
        if (tid == 0)
            a.mb_rowoff0[i] = row0;
        if (last && tid == 0)
            a.mb_rowoff0[a.k] = row0 + a.b;
        __syncthreads();
        for (int32_t j = tid; j < a.b; j += kSmThreads) {
            const int32_t v = a.batches[row0 + j];
            a.row_vertex0[row0 + j] = v;
            if (v < 0 || (int64_t)v >= a.n) {
                a.seed_flags[0] = 1;
                continue;
            }
            uint32_t slot = ((uint32_t)v * 0x9E3779B1u) >> a.seed_shift;
            while (true) {
                const uint32_t old = atomicCAS(&key[slot], kSmEmpty, (uint32_t)v);
                if (old == kSmEmpty)
                    break;
                if (old == (uint32_t)v) {
                    a.seed_flags[1] = 1;
                    break;
                }
                slot = (slot + 1u) & (uint32_t)(slots - 1);
            }
        }
        __syncthreads();
    }

    const int32_t *rows = a.row_vertex0 + row0;
    int64_t rows_total = (int64_t)a.k * a.b; // (of the last minibatch only)
    for (int32_t h = 0; h < a.nhops; ++h) {
        const NwSmallHop &H = a.hop[h];
        const uint32_t mb = a.mb_base + (uint32_t)i;
        int64_t *rowptr = H.rowptr + row0;
        int32_t nnz;
        if (H.s <= 4)
            nnz = small_sample_rows<4, REPLACE>(a, H.hopkey, H.s, mb, rows, R, rowptr, key, wsum);
        else if (H.s <= 8)
            nnz = small_sample_rows<8, REPLACE>(a, H.hopkey, H.s, mb, rows, R, rowptr, key, wsum);
        else if (SMAX == 16 || H.s <= 16)
            nnz = small_sample_rows<16, REPLACE>(a, H.hopkey, H.s, mb, rows, R, rowptr, key, wsum);
        else
            nnz = small_sample_rows<SMAX, REPLACE>(a, H.hopkey, H.s, mb, rows, R, rowptr, key, wsum);
        const int32_t self = a.self_entry ? R : 0; // entries [0, self): the rows' own vertices, then the sampled ones
        const int32_t N = nnz + self;
        __syncthreads();

        // sorted order of the entries by id: by[x] = position of the x-th smallest.  Every wave owns `per` consecutive
        // places, 64 of them in each of its steps
        const int32_t per = ((N + kSmWaves - 1) / kSmWaves + kWave - 1) / kWave * kWave;
        const int32_t e0 = wave * per, e1 = min(e0 + per, N);
        uint16_t *by = small_sort_buckets(a, key, pos, pos + a.cap, work, N, wsum, &crowded_s);
        if (!by)
            by = small_sort_radix(a.idbits, key, pos, pos + a.cap, work, N, e0, e1, wave, wsum);
        uint16_t *rank_of = by == pos ? pos + a.cap : pos; // the other array is free

        // heads of the runs of equal ids, one mask per step
        unsigned long long *mask = reinterpret_cast<unsigned long long *>(work);
        uint32_t heads = 0; // of this wave's part
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
        uint32_t before = 0, U = 0;
#pragma unroll
        for (int w = 0; w < kSmWaves; ++w) {
            before += w < wave ? wsum[w] : 0u;
            U += wsum[w];
        }
        // sizes of this minibatch for everyone after it
        unsigned long long *status = a.status + (int64_t)h * a.k;
        if (tid == 0)
            __hip_atomic_store(status + i, ((unsigned long long)a.epoch << 32) | ((unsigned long long)(uint32_t)nnz << 16) | U,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // local columns by position
        uint32_t run = before;
        for (int32_t eb = e0; eb < e1; eb += kWave) {
            const uint64_t hm = mask[eb / kWave];
            if (eb + lane < e1)
                rank_of[by[eb + lane]] = (uint16_t)(run + (uint32_t)__popcll(hm & (below | (1ull << lane))) - 1u);
            run += (uint32_t)__popcll(hm);
        }
        // entries, columns and row tiles of the minibatches before this one
        int64_t sum_e = 0, sum_c = 0, sum_t = 0;
        int32_t most = (int32_t)((U + kRowTile - 1) / kRowTile);
        for (int32_t j = tid; j < i; j += kSmThreads) {
            unsigned long long w;
            while ((uint32_t)((w = __hip_atomic_load(status + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> 32) != a.epoch)
                __builtin_amdgcn_s_sleep(2);
            const int32_t cols = (int32_t)(w & 0xFFFFu), tiles = (cols + kRowTile - 1) / kRowTile;
            sum_e += (int64_t)((w >> 16) & 0xFFFFu);
            sum_c += cols;
            sum_t += tiles;
            most = tiles > most ? tiles : most;
        }
        int64_t total;
        (void)block_exclusive_scan<int64_t, kSmThreads>(sum_e, wsum64, total);
        const int64_t edge0 = total;
        (void)block_exclusive_scan<int64_t, kSmThreads>(sum_c, wsum64, total);
        const int64_t col0 = total;
        __syncthreads();

        for (int32_t r = tid; r < R; r += kSmThreads)
            rowptr[r] += edge0; // written by this thread
        for (int32_t e = tid; e < nnz; e += kSmThreads)
            H.col[edge0 + e] = (int32_t)rank_of[self + e];
        for (int32_t r = tid; r < self; r += kSmThreads)
            H.row_self[row0 + r] = (int32_t)rank_of[r];
        run = before;
        for (int32_t eb = e0; eb < e1; eb += kWave) {
            const uint64_t hm = mask[eb / kWave];
            if ((hm >> lane) & 1ull)
                H.col_vertex[col0 + run + (uint32_t)__popcll(hm & below)] = (int32_t)key[by[eb + lane]];
            run += (uint32_t)__popcll(hm);
        }
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
        if (h == a.nhops - 1 && a.next_tileoff) { // row tiles of the hop that follows on the chip-wide path
            (void)block_exclusive_scan<int64_t, kSmThreads>(sum_t, wsum64, total);
            if (tid == 0)
                a.next_tileoff[i] = total;
            if (last) {
                const int64_t tiles_before = total;
#pragma unroll
                for (int d = kWave / 2; d > 0; d >>= 1)
                    most = max(most, __shfl_xor(most, d, kWave));
                __syncthreads();
                if (lane == 0)
                    wsum[wave] = (uint32_t)most;
                __syncthreads();
                if (tid == 0) {
                    for (int w = 0; w < kSmWaves; ++w)
                        most = max(most, (int32_t)wsum[w]);
                    a.next_tileoff[a.k] = tiles_before + (U + kRowTile - 1) / kRowTile;
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
        rows = H.col_vertex + col0;
        row0 = col0;
        R = (int32_t)U;
        __syncthreads(); // the next frontier is in memory for every wave of this workgroup; LDS is free
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
