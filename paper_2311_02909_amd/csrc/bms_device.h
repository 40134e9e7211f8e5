// Device-side building blocks shared by the sampler kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bms {

constexpr int kWave = 64;
constexpr int kRowTile = 256;      // stacked rows handled by one workgroup iteration (one row per lane)
constexpr int kLineWords = 16;     // a vertex-set "line": 16 x 32-bit words = 512 vertex ids = 64 bytes
constexpr int kLineBits = 512;
constexpr int kChunkLines = 256;   // lines ranked by one workgroup (131072 vertex ids)

// T in device memory.  A pointer that was computed as a number, or comes from LDS, is not known to lead there: its loads count as
// accesses of LDS too, and every later access of LDS waits for all of them.
template <class T>
using Global = __attribute__((address_space(1))) T;
using U32x4 = uint32_t __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------------------------
// Counter-based random stream: a stateless hash of (seed, hop, minibatch, vertex, draw index).
// 64-bit work happens once per distribution (the key); every draw is 32-bit arithmetic.
// ---------------------------------------------------------------------------------------------
__host__ __device__ inline uint64_t mix64(uint64_t x)
{
    x ^= x >> 30;
    x *= 0xBF58476D1CE4E5B9ULL;
    x ^= x >> 27;
    x *= 0x94D049BB133111EBULL;
    x ^= x >> 31;
    return x;
}

__host__ __device__ inline uint32_t fin32(uint32_t x)
{
    x ^= x >> 16;
    x *= 0x7FEB352DU;
    x ^= x >> 15;
    x *= 0x846CA68BU;
    x ^= x >> 16;
    return x;
}

// key of the (seed, hop) pair; computed on the host once per hop
__host__ __device__ inline uint64_t hop_key(uint64_t seed, int32_t hop)
{
    return mix64(seed ^ (0x9E3779B97F4A7C15ULL * (uint64_t)(hop + 1)));
}

__host__ __device__ inline uint64_t row_key(uint64_t hopkey, uint32_t mb, uint32_t vertex)
{
    return mix64(hopkey ^ (((uint64_t)mb << 32) | (uint64_t)vertex));
}

__device__ inline uint32_t draw32(uint64_t key, uint32_t j)
{
    return fin32(fin32((uint32_t)key + j * 0x9E3779B9U) ^ (uint32_t)(key >> 32));
}

__device__ inline uint64_t draw64(uint64_t key, uint32_t j)
{
    return ((uint64_t)draw32(key, 2u * j) << 32) | (uint64_t)draw32(key, 2u * j + 1u);
}

__device__ inline uint32_t bounded32(uint32_t x, uint32_t m) { return __umulhi(x, m); }
__device__ inline uint64_t bounded64(uint64_t x, uint64_t w) { return __umul64hi(x, w); }

constexpr uint32_t kNoVertex = 0xFFFFFFFFu;

// Sums over the workgroups before one's own, inside a launch (take_number, sum_before): at most kMostLookback workgroups
constexpr int kMostLookback = 1024;
struct Lookback {
    unsigned long long *status; // kMostLookback words: epoch << 40 | value
    uint32_t *ticket;           // device counter: workgroups that have started
    uint32_t ticket0;           // its value before the launch
    uint32_t epoch;             // of the launch, 24 bits, never 0
};

// ---------------------------------------------------------------------------------------------
// Scans
// ---------------------------------------------------------------------------------------------
template <class T>
__device__ inline T wave_inclusive_scan(T v)
{
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        T o = __shfl_up(v, d, kWave);
        if (lane >= d)
            v += o;
    }
    return v;
}

// The same for 32-bit counts through the vector unit's lane-permute paths only (no LDS crossbar): shifts inside
// each row of 16 lanes, then the last lane of rows 0 and 2 broadcast into rows 1 and 3, then lane 31 into rows 2, 3.
__device__ inline uint32_t wave_inclusive_scan_dpp(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111 /* row_shr:1 */, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112 /* row_shr:2 */, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114 /* row_shr:4 */, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118 /* row_shr:8 */, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142 /* row_bcast:15 */, 0xA, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143 /* row_bcast:31 */, 0xC, 0xF, false);
    return v;
}

template <class T>
__device__ inline T wave_sum(T v)
{
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1)
        v += __shfl_xor(v, d, kWave);
    return v;
}

// 64-lane bitonic sorting network, ascending by lane
__device__ inline uint32_t wave_sort_u32(uint32_t c, int lane)
{
#pragma unroll
    for (int kk = 2; kk <= kWave; kk <<= 1) {
#pragma unroll
        for (int j = kk >> 1; j > 0; j >>= 1) {
            const uint32_t o = __shfl_xor(c, j, kWave);
            const bool keep_min = ((lane & j) == 0) == ((lane & kk) == 0);
            c = keep_min ? min(c, o) : max(c, o);
        }
    }
    return c;
}

// Exclusive scan over the NT threads of a workgroup.  `smem` holds NT/64 values of T.
// Contains two barriers; smem may be reused after the call returns on all threads
// only after another barrier (the callers loop with barriers in between).
template <class T, int NT>
__device__ inline T block_exclusive_scan(T v, T *smem, T &total)
{
    constexpr int NW = NT / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    T inc = wave_inclusive_scan(v);
    __syncthreads(); // protects smem against readers of a previous call
    if (lane == kWave - 1)
        smem[wave] = inc;
    __syncthreads();
    T before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        T x = smem[w];
        if (w < wave)
            before += x;
        all += x;
    }
    total = all;
    return before + inc - v;
}

// A value that is the same in all of a wave's lanes, in scalar registers.  The compiler does not see it of values loaded from
// memory that the kernel writes to, or that follow from the wave's number, and keeps a copy of them in every lane.
__device__ inline int64_t lane_value(int64_t x, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)x >> 32), lane);
    return (int64_t)((uint64_t)hi << 32 | lo);
}
__device__ inline uint32_t scalar(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ inline int64_t scalar(int64_t x)
{
    return (int64_t)((uint64_t)scalar((uint32_t)((uint64_t)x >> 32)) << 32 | scalar((uint32_t)x));
}

// A value read at an address that is the same in all lanes, of an array that nothing writes during the launch: through the
// scalar unit, which the compiler does not choose by itself when the kernel writes to other arrays.
template <class T>
__device__ inline T uniform_load(const T *p)
{
    return *(const __attribute__((address_space(4))) T *)(uintptr_t)p;
}

// Bits of `mask` below the lane's own, without a mask of them in registers
__device__ inline uint32_t bits_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Entries v and v + 1 of a CSR's row pointers in one read (8-byte aligned)
using int64x2_a8 = int64_t __attribute__((ext_vector_type(2), aligned(8)));
__device__ inline int64x2_a8 row_extent(const int64_t *rowptr, int64_t v)
{
    return *reinterpret_cast<const int64x2_a8 *>(rowptr + v);
}

// A workgroup's number in its launch, in the order of starting: whoever waits for lower numbers waits for workgroups that
// have started.  smem: one word of LDS.
__device__ inline uint32_t take_number(const Lookback &lb, uint32_t *smem)
{
    if (threadIdx.x == 0)
        *smem = atomicAdd(lb.ticket, 1u) - lb.ticket0;
    __syncthreads();
    return *smem;
}

// Sum of the values that workgroups 0 .. i - 1 of the launch bring, for workgroup number i, which brings `value` (below 2^40);
// all threads of the workgroup call it.  Every workgroup leaves its value before it waits for anyone.
template <int NT>
__device__ inline int64_t sum_before(const Lookback &lb, uint32_t i, int64_t value, int64_t *smem /* NT / 64 */)
{
    if (threadIdx.x == 0)
        __hip_atomic_store(lb.status + i, ((unsigned long long)lb.epoch << 40) | (unsigned long long)value, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    int64_t sum = 0;
    for (uint32_t j = threadIdx.x; j < i; j += NT) {
        unsigned long long w;
        while ((uint32_t)((w = __hip_atomic_load(lb.status + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> 40) != lb.epoch)
            __builtin_amdgcn_s_sleep(1);
        sum += (int64_t)(w & ((1ull << 40) - 1ull));
    }
    sum = wave_sum(sum);
    __syncthreads();
    if ((threadIdx.x & (kWave - 1)) == 0)
        smem[threadIdx.x / kWave] = sum;
    __syncthreads();
    sum = 0;
#pragma unroll
    for (int w = 0; w < NT / kWave; ++w)
        sum += smem[w];
    return sum;
}

// One thread of every workgroup of a launch, after its atomic stores of what the last one is to read: true for the one that
// comes here last.  *done is zero before and after.
__device__ inline bool arrive_last(uint32_t *done, uint32_t workgroups)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // what was stored is where other dies see it
    if (__hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != workgroups - 1u)
        return false;
    __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

// Called by all threads of each of a launch's `parts` workgroups when the workgroup has written everything: the last of
// them writes `arrival` to *arrived, in host memory, behind all the writes.  *done is zero before and after.
__device__ inline void announce(uint32_t *done, uint32_t parts, int64_t *arrived, int64_t arrival)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // every wave's writes have left it; one thread then releases them all
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence_system();
        if (__hip_atomic_fetch_add(done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == parts - 1u) {
            __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(arrived, arrival, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// Minibatch i's b seeds by a workgroup of NT threads: copied (copy not null), and passed through a hash table of `slots` words in LDS, a power of two
// >= 2 b, shift = 32 - its log2; flags[0]: one lies outside [0, n), flags[1]: one is repeated.
template <int NT>
__device__ inline void check_seeds(const int32_t *seeds, int i, int32_t b, int64_t n, int32_t slots, int32_t shift, uint32_t *key,
                                   int32_t *copy, int32_t *flags)
{
    const int tid = threadIdx.x;
    const int64_t row0 = (int64_t)i * b;
    for (int32_t x = tid; x < slots; x += NT)
        key[x] = 0xFFFFFFFFu;
    __syncthreads();
    for (int32_t j = tid; j < b; j += NT) {
        const int32_t v = seeds[row0 + j];
        if (copy)
            copy[row0 + j] = v;
        if (v < 0 || (int64_t)v >= n) {
            flags[0] = 1;
            continue;
        }
        uint32_t slot = ((uint32_t)v * 0x9E3779B1u) >> shift;
        while (true) {
            const uint32_t old = atomicCAS(&key[slot], 0xFFFFFFFFu, (uint32_t)v);
            if (old == 0xFFFFFFFFu)
                break;
            if (old == (uint32_t)v) {
                flags[1] = 1;
                break;
            }
            slot = (slot + 1u) & (uint32_t)(slots - 1);
        }
    }
}

// Largest i in [0,k) with off[i] <= t, given off[0] <= t < off[k] (off ascending, k >= 1).
__device__ inline int locate_segment(const int64_t *__restrict__ off, int k, int64_t t)
{
    int lo = 0, hi = k;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (off[mid] <= t)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// The same through the scalar unit: off is not written during the launch, t the same in all lanes.
__device__ inline int locate_uniform(const int64_t *off, int k, int64_t t)
{
    int lo = 0, hi = k;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (uniform_load(off + mid) <= t)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// Rank of vertex g inside one minibatch's vertex set: set bits before it = line_prefix of its
// 64-byte line + set bits before it inside the line.  `words`/`line_prefix` point at the
// minibatch's own slice.
__device__ inline int32_t vset_rank_of(const uint32_t *__restrict__ words, const uint32_t *__restrict__ line_prefix,
                                       int32_t g)
{
    const int32_t line = g >> 9;
    const int32_t w = (g >> 5) & (kLineWords - 1);
    const uint4 *p = reinterpret_cast<const uint4 *>(words + (int64_t)line * kLineWords);
    uint32_t rank = line_prefix[line];
    const int nq = w >> 2; // whole 16-byte quarters before the word
    for (int q = 0; q < nq; ++q) {
        const uint4 x = p[q];
        rank += __popc(x.x) + __popc(x.y) + __popc(x.z) + __popc(x.w);
    }
    const uint4 x = p[nq];
    const uint32_t xs[4] = {x.x, x.y, x.z, x.w};
    const int rem = w & 3;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (q < rem)
            rank += __popc(xs[q]);
        else if (q == rem)
            rank += __popc(xs[q] & ((1u << (g & 31)) - 1u));
    }
    return (int32_t)rank;
}

__device__ inline bool vset_test(const uint32_t *__restrict__ words, int32_t g)
{
    return (words[g >> 5] >> (g & 31)) & 1u;
}

} // namespace bms
