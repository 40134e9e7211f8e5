// EXTRACT for the node-wise sampler over vertex ranges (Sec. 4.1.3: "remove empty columns"): the distinct sampled ids of a
// minibatch as one bit per vertex, the rank of an id = set bits before it.
//
// A bitmap of [0, n) takes n / 8 bytes per minibatch, too much for LDS at once, so it is worked on in ranges of ids:
//   mark     per (minibatch, range of up to 1.28 million ids): the minibatch's ids stream by, those inside the range set their
//            bit in LDS; then set bits are counted per quad (128 ids), and quads and counts leave for memory.  Where
//            minibatches and ranges are too few to fill the chip, the entries are shared by several workgroups, the bitmaps
//            leave as they are and `count` merges and counts them.  Few minibatches (at most kRangesFewMb): the sampling
//            kernel sets the bits in memory itself
//   count    see above.  The workgroup of mark or count that ends last turns the counts of all ranges into where each
//            begins in the stacked columns: column offsets, the next hop's row tiles
//   emit     the set bits as ids in ascending order = the next frontier, staged through LDS, written coalesced
//   lookup   per chunk of up to 57344 entries of a minibatch, held in registers: for one range of ids after the other
//            the (32 bits, set bits before them) words go to LDS and the ids inside the range become local columns, in place;
//            few entries: each entry's word is fetched by itself (gather, in the same launch as emit)
//
// Against the cut into segments (kernels_dedup_sort.hip: per entry 30 bytes and 12 per distinct id moved in runs, 9
// launches a hop) the ids are read twice and written once, in 6 launches, 5 for few entries.  What bounds mark and lookup
// are the instructions per entry and range (about 10, however few of 64 ids are inside the range).  The work
// grows with the number of ranges, so this is the path of graphs of a few million vertices (ranges_apply in bms_api.hip).
// Measured on the last hop of 64 x 1024 seeds, (15, 10, 5), 2.4 M vertices (27.9 M entries, 18.8 M columns): mark 50, emit 22,
// lookup 73 us where the cut took 288 us; 8 minibatches 61 and 82 us, one (442 k entries) 22 and 66 when they were compared (5 to
// 10 us less on this side since).
// With BMS_UNION_DST the frontier's own vertices are marked and looked up as well, straight from the frontier: rows carry
// no extra entry.
#include "bms_device.h"
#include "bms_internal.h"

#include <algorithm>

namespace bms {

constexpr int kRgThreads = 1024;
constexpr int kRgWaves = kRgThreads / kWave;
constexpr int kMarkQuads = 9984;  // of a mark workgroup, at most: 156 KB
constexpr int kMarkIts = 9;       // quads per lane of one that counts, at most
constexpr int kMarkUnroll = 4;    // 16-byte loads in flight per lane
constexpr int kMarkRows = 8;      // 4-byte loads
constexpr int kMostParts = 32;
constexpr int kTableQuads = 4864; // quads of a lookup table: 4 words of 8 bytes each, 152 KB
constexpr int kTablePer = (kTableQuads + kRgThreads - 1) / kRgThreads;
constexpr int kEmitQuads = 16; // quads per step of a wave of emit: 2048 ids, 4 KB of 16-bit places
static_assert(kEmitQuads * 4 == kWave && kRangeQuads % kRgThreads == 0 && kRgThreads % kEmitQuads == 0, "steps out of step");

__device__ inline uint32_t quad_popc(const uint4 &q) { return __popc(q.x) + __popc(q.y) + __popc(q.z) + __popc(q.w); }

// range of a quad: exact, as quads * qw < 2^32 unless qw is a power of two
__device__ inline uint32_t range_of(const RangeArgs &a, uint32_t quad) { return __umulhi(quad, a.qw_inverse); }

// The counts of all (minibatch, range) pairs are in a.cnt; run by one workgroup of NT threads, which everything after it waits
// for.  room: NT + 1 words of LDS.
// Up to NT pairs without going through memory and in 32 bits (a range has no more than 1.3 million ids): 6 us of a hop before, 1.5 so (count
// kernel of one minibatch 10 -> 5.2 us, mark kernels 3 to 5 us less).
template <int NT>
__device__ inline void ranges_place(const RangeArgs &a, uint32_t *room)
{
    __shared__ int64_t smem[NT / kWave];
    __shared__ int32_t most_s;
    const int tid = threadIdx.x;
    const int64_t m = (int64_t)a.k * a.H;
    if (m <= NT) {
        uint32_t *wsum = reinterpret_cast<uint32_t *>(smem); // two sums per wave
        const int lane = tid & (kWave - 1), wave = tid / kWave;
        // exclusive scan, the total; half: which of the two words per wave
        auto scan = [&](uint32_t v, int half, uint32_t &total) {
            const uint32_t upto = wave_inclusive_scan_dpp(v);
            if (lane == kWave - 1)
                wsum[half * (NT / kWave) + wave] = upto;
            __syncthreads();
            uint32_t before = 0;
            total = 0;
#pragma unroll
            for (int x = 0; x < NT / kWave; ++x) {
                const uint32_t sum = wsum[half * (NT / kWave) + x];
                before += x < wave ? sum : 0u;
                total += sum;
            }
            return before + upto - v;
        };
        if (tid == 0)
            most_s = 0;
        const uint32_t v = tid < m ? __hip_atomic_load(a.cnt + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        uint32_t columns, tiles_all;
        const uint32_t ex = scan(v, 0, columns);
        room[tid] = ex;
        if (tid == 0)
            room[NT] = columns;
        __syncthreads();
        uint32_t tiles = 0, c0 = 0;
        if (tid < a.k) {
            c0 = room[tid * a.H];
            tiles = (room[tid + 1 < a.k ? (tid + 1) * a.H : NT] - c0 + kRowTile - 1) / kRowTile;
            atomicMax(&most_s, (int32_t)tiles);
        }
        const uint32_t tile0 = scan(tiles, 1, tiles_all);
        if (tid < m)
            a.first[tid] = ex;
        if (tid < a.k) {
            a.mb_coloff[tid] = c0;
            a.next_tileoff[tid] = tile0;
        }
        if (tid == 0) {
            a.first[m] = columns;
            a.mb_coloff[a.k] = columns;
            *a.ncols_out = columns;
            a.next_tileoff[a.k] = tiles_all;
            a.next_tileoff[a.k + 1] = most_s;
        }
        return;
    }
    int64_t carry = 0;
    for (int64_t base = 0; base < m; base += NT) {
        const int64_t x = base + tid;
        const int64_t v = x < m ? (int64_t)__hip_atomic_load(a.cnt + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
        int64_t total;
        const int64_t ex = carry + block_exclusive_scan<int64_t, NT>(v, smem, total);
        if (x < m) {
            a.first[x] = ex;
            if (x % a.H == 0)
                a.mb_coloff[x / a.H] = ex;
        }
        carry += total;
    }
    if (tid == 0) {
        a.first[m] = carry;
        a.mb_coloff[a.k] = carry;
        *a.ncols_out = carry;
        most_s = 0;
    }
    __syncthreads(); // mb_coloff was written by this workgroup
    int64_t tiles_before = 0;
    int32_t most = 0;
    for (int32_t base = 0; base < a.k; base += NT) {
        const int32_t i = base + tid;
        int64_t tiles = 0;
        if (i < a.k)
            tiles = (a.first[(int64_t)(i + 1) * a.H] - a.first[(int64_t)i * a.H] + kRowTile - 1) / kRowTile;
        most = max(most, (int32_t)tiles);
        int64_t total;
        const int64_t ex = tiles_before + block_exclusive_scan<int64_t, NT>(tiles, smem, total);
        if (i < a.k)
            a.next_tileoff[i] = ex;
        tiles_before += total;
    }
    atomicMax(&most_s, most);
    __syncthreads();
    if (tid == 0) {
        a.next_tileoff[a.k] = tiles_before;
        a.next_tileoff[a.k + 1] = most_s;
    }
}

// One thread of every workgroup of the launch: leaves the workgroup's count for the one that comes here last (true).
__device__ inline bool count_arrives(uint32_t *cnt, uint32_t count, uint32_t *done, uint32_t workgroups)
{
    __hip_atomic_store(cnt, count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return arrive_last(done, workgroups);
}

// Workgroups go to the chip's 8 dies in turn.  Of a launch with `per` workgroups for every minibatch, those of one minibatch
// sit on one die (whose L2 then serves the ids or tables that they share), except in the last group of fewer than 8
// minibatches: workgroup b is number `x` of minibatch `i`.
__device__ inline void die_order(uint32_t b, uint32_t k, uint32_t per, int &i, uint32_t &x)
{
    const uint32_t group = b / (8u * per), in_group = b - group * 8u * per;
    const uint32_t mbs = min(8u, k - 8u * group);
    i = (int)(8u * group + in_group % mbs);
    x = in_group / mbs;
}

// set bits before each of the `its` x 64 consecutive quads of a wave and the total of the workgroup; wtot: one word per wave
template <int MOST, class Get>
__device__ inline uint32_t count_quads(int its, uint32_t *wtot, uint32_t (&before)[MOST], Get get)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    uint32_t wave_total = 0;
#pragma unroll
    for (int it = 0; it < MOST; ++it) {
        before[it] = 0;
        if (it < its) {
            const uint32_t pc = quad_popc(get(it));
            const uint32_t inc = wave_inclusive_scan_dpp(pc) + wave_total;
            before[it] = inc - pc;
            wave_total = (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
        }
    }
    if (lane == 0)
        wtot[wave] = wave_total;
    __syncthreads();
    uint32_t run = 0, total = 0;
#pragma unroll
    for (int x = 0; x < kRgWaves; ++x) {
        run += x < wave ? wtot[x] : 0u;
        total += wtot[x];
    }
#pragma unroll
    for (int it = 0; it < MOST; ++it)
        before[it] += run;
    return total;
}

// Ranges of mq quads.  COUNT: mq = a.qw, one part.  Else the bitmap of part p of minibatch i goes to bits + (p k + i) stride.
template <bool COUNT>
__global__ __launch_bounds__(kRgThreads) void rg_mark_kernel(RangeArgs a, int32_t mq)
{
    extern __shared__ uint4 mark_lds[]; // mq quads
    __shared__ uint32_t wtot[kRgWaves];
    __shared__ uint32_t last_s;
    const int tid = threadIdx.x;
    int i;
    uint32_t x;
    die_order(blockIdx.x, (uint32_t)a.k, gridDim.x / (uint32_t)a.k, i, x);
    const int w = (int)(x / (uint32_t)a.parts), part = (int)(x % (uint32_t)a.parts);
    uint32_t *words = reinterpret_cast<uint32_t *>(mark_lds);
    for (int q = tid; q < mq; q += kRgThreads)
        mark_lds[q] = make_uint4(0, 0, 0, 0);
    const uint32_t lo = (uint32_t)w * (uint32_t)mq * 128u;
    const uint32_t ids = (uint32_t)min((int64_t)mq * 128, a.n - (int64_t)lo); // of this range
    const int64_t r0 = a.mb_rowoff[i], r1 = a.mb_rowoff[i + 1];
    const int64_t all0 = a.rowptr[r0], all1 = a.rowptr[r1];
    const int64_t per = ((all1 - all0 + a.parts - 1) / a.parts + 3) & ~(int64_t)3;
    const int64_t e0 = min(all0 + part * per, all1), e1 = min(e0 + per, all1);
    __syncthreads();
    auto mark = [&](uint32_t id) {
        const uint32_t rel = id - lo;
        if (rel < ids)
            atomicOr(&words[rel >> 5], 1u << (rel & 31u));
    };
    // the entries before the first whole 16 bytes, the whole ones, the entries after them
    const int32_t *__restrict__ col = a.col;
    const int64_t b0 = min((e0 + 3) & ~(int64_t)3, e1), b1 = max(e1 & ~(int64_t)3, b0);
    if (tid < (int)(b0 - e0))
        mark((uint32_t)col[e0 + tid]);
    if (tid < (int)(e1 - b1))
        mark((uint32_t)col[b1 + tid]);
    const uint4 *__restrict__ col4 = reinterpret_cast<const uint4 *>(col);
    const int64_t c1 = b1 >> 2;
    // Whole steps of the workgroup two by two, each one's 16-byte loads on their way while the other's ids are marked (no
    // lane is ever without a load, so nothing but the uses waits for them); then what is left.
    const int64_t cb = (b0 >> 2) + tid;
    const int64_t steps = (c1 - (b0 >> 2)) / (kMarkUnroll * kRgThreads);
    uint4 va[kMarkUnroll], vb[kMarkUnroll];
    auto fetch = [&](int64_t step, uint4 (&v)[kMarkUnroll]) {
#pragma unroll
        for (int u = 0; u < kMarkUnroll; ++u)
            v[u] = col4[cb + (step * kMarkUnroll + u) * kRgThreads];
    };
    auto mark_all = [&](const uint4 (&v)[kMarkUnroll]) {
#pragma unroll
        for (int u = 0; u < kMarkUnroll; ++u) {
            mark(v[u].x);
            mark(v[u].y);
            mark(v[u].z);
            mark(v[u].w);
        }
    };
    if (steps > 0)
        fetch(0, va);
    for (int64_t step = 0; step < steps; step += 2) {
        if (step + 1 < steps)
            fetch(step + 1, vb);
        mark_all(va);
        if (step + 2 < steps)
            fetch(step + 2, va);
        if (step + 1 < steps)
            mark_all(vb);
    }
    for (int64_t c0 = cb + steps * kMarkUnroll * kRgThreads; c0 < c1; c0 += kRgThreads) {
        const uint4 v = col4[c0];
        mark(v.x);
        mark(v.y);
        mark(v.z);
        mark(v.w);
    }
    if (a.row_self)
        for (int64_t c = r0 + part * kRgThreads + tid; c < r1; c += (int64_t)a.parts * kMarkRows * kRgThreads) {
            uint32_t id[kMarkRows]; // in flight together
#pragma unroll
            for (int u = 0; u < kMarkRows; ++u) {
                const int64_t r = c + (int64_t)u * a.parts * kRgThreads;
                id[u] = r < r1 ? (uint32_t)a.row_vertex[r] : ~0u; // (no id)
            }
#pragma unroll
            for (int u = 0; u < kMarkRows; ++u)
                mark(id[u]);
        }
    __syncthreads();
    if (COUNT) {
        const int its = mq / kRgThreads, wave_quad = (tid / kWave) * its * kWave + (tid & (kWave - 1));
        uint32_t before[kMarkIts];
        const uint32_t total = count_quads<kMarkIts>(its, wtot, before, [&](int it) { return mark_lds[wave_quad + it * kWave]; });
        if (tid == 0) // before the stores below: the workgroup's turn is known when they are done
            last_s = count_arrives(a.cnt + (int64_t)i * a.H + w, total, a.done, (uint32_t)gridDim.x) ? 1u : 0u;
        const int64_t q0 = (int64_t)i * a.stride + (int64_t)w * mq + wave_quad;
#pragma unroll
        for (int it = 0; it < kMarkIts; ++it)
            if (it < its) {
                a.bits[q0 + it * kWave] = mark_lds[wave_quad + it * kWave];
                a.pre[q0 + it * kWave] = before[it];
            }
        __syncthreads();
        if (last_s)
            ranges_place<kRgThreads>(a, words); // (the bitmap has left)
        return;
    }
    uint4 *__restrict__ out = a.bits + ((int64_t)part * a.k + i) * a.stride;
    const int q0 = w * mq, q1 = (int)min<int64_t>((int64_t)q0 + mq, a.stride);
    for (int q = q0 + tid; q < q1; q += kRgThreads)
        out[q] = mark_lds[q - q0];
    if (q1 >= (int)a.quads) // the last range: what rounds the minibatch's bitmap up
        for (int64_t q = q1 + tid; q < a.stride; q += kRgThreads)
            out[q] = make_uint4(0, 0, 0, 0);
}

// Parts merged, set bits before every quad.  One workgroup per (minibatch, range of kRangeQuads quads): blockIdx.x = range * k
// + minibatch.
__global__ __launch_bounds__(kRgThreads) void rg_count_kernel(RangeArgs a)
{
    constexpr int ITS = kRangeQuads / kRgThreads;
    __shared__ uint32_t wtot[kRgWaves], room[kRgThreads + 1];
    __shared__ uint32_t last_s;
    const int tid = threadIdx.x;
    const int i = (int)(blockIdx.x % (uint32_t)a.k), w = (int)(blockIdx.x / (uint32_t)a.k);
    const int64_t q0 = (int64_t)i * a.stride + (int64_t)w * kRangeQuads + (tid / kWave) * (ITS * kWave) + (tid & (kWave - 1));
    uint4 v[ITS];
#pragma unroll
    for (int it = 0; it < ITS; ++it)
        v[it] = a.bits[q0 + it * kWave];
    for (int32_t p = 1; p < a.parts; ++p) {
        const uint4 *__restrict__ more = a.bits + (int64_t)p * a.k * a.stride + q0;
#pragma unroll
        for (int it = 0; it < ITS; ++it) {
            const uint4 x = more[it * kWave];
            v[it] = make_uint4(v[it].x | x.x, v[it].y | x.y, v[it].z | x.z, v[it].w | x.w);
        }
    }
    uint32_t before[ITS];
    const uint32_t total = count_quads<ITS>(ITS, wtot, before, [&](int it) { return v[it]; });
    if (tid == 0)
        last_s = count_arrives(a.cnt + (int64_t)i * a.H + w, total, a.done, (uint32_t)gridDim.x) ? 1u : 0u;
#pragma unroll
    for (int it = 0; it < ITS; ++it) {
        if (a.parts > 1)
            a.bits[q0 + it * kWave] = v[it];
        a.pre[q0 + it * kWave] = before[it];
    }
    __syncthreads();
    if (last_s)
        ranges_place<kRgThreads>(a, room);
}

// Set bits -> ids, wave x of nx: steps of kEmitQuads quads of a minibatch, a word per lane.  The set bits before a quad are known,
// so a wave needs no other and waits for none.  places: LDS of this wave, kEmitQuads * 128 16-bit values.
// Half vector instructions (100 per step and ten per round of bits), half the step's own chain.  Two hops of 64 x 1024 seeds, (15,
// 10, 5), 2.4 M vertices: 54 us by workgroups of 1024 in steps of 32768 ids with three barriers, 38.5 so;
// eighths of the steps per die, or the range's first column fetched a step ahead, change nothing.
__device__ inline void emit_steps(const RangeArgs &a, int32_t *__restrict__ col_vertex, uint16_t *places, uint32_t x, uint32_t nx)
{
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t steps = (uint32_t)((a.quads + kEmitQuads - 1) / kEmitQuads); // per minibatch
    const uint32_t *__restrict__ words = reinterpret_cast<const uint32_t *>(a.bits);
    uint32_t word = 0, pre = 0, word_next = 0, pre_next = 0;
    auto fetch = [&](uint32_t i, uint32_t step, uint32_t &wd, uint32_t &p) {
        if (i < (uint32_t)a.k) {
            const int64_t q = i * a.stride + (int64_t)step * kEmitQuads;
            wd = (words + q * 4)[lane];
            p = (a.pre + q)[lane >> 2];
        }
    };
    uint32_t i = x / steps, step = x % steps;
    const uint32_t more_i = nx / steps, more_step = nx % steps;
    fetch(i, step, word, pre);
    while (i < (uint32_t)a.k) {
        uint32_t i_next = i + more_i, step_next = step + more_step;
        if (step_next >= steps) {
            step_next -= steps;
            ++i_next;
        }
        fetch(i_next, step_next, word_next, pre_next);
        const int64_t first = uniform_load(a.first + (int64_t)i * a.H + range_of(a, step * kEmitQuads));
        // set bits of the quad's words before this one
        const int pc = __popc(word);
        const int back1 = __builtin_amdgcn_update_dpp(0, pc, 0x90 /* quad_perm:[0,0,1,2] */, 0xF, 0xF, true);
        const int back2 = __builtin_amdgcn_update_dpp(0, pc, 0x40 /* quad_perm:[0,0,0,1] */, 0xF, 0xF, true);
        const int back3 = __builtin_amdgcn_update_dpp(0, pc, 0x00 /* quad_perm:[0,0,0,0] */, 0xF, 0xF, true);
        const int lower = ((lane & 3) >= 1 ? back1 : 0) + ((lane & 3) >= 2 ? back2 : 0) + ((lane & 3) >= 3 ? back3 : 0);
        const uint32_t p0 = scalar(pre);
        uint32_t at = pre + (uint32_t)lower - p0;
        const uint32_t count = (uint32_t)__builtin_amdgcn_readlane((int)(at + (uint32_t)pc), kWave - 1);
        for (uint32_t wd = word; wd; wd &= wd - 1u)
            places[at++] = (uint16_t)(lane * 32 + (__ffs((int)wd) - 1));
        __builtin_amdgcn_wave_barrier();
        int32_t *__restrict__ out = col_vertex + first + p0;
        const int32_t id0 = (int32_t)(step * kEmitQuads * 128u);
        for (uint32_t j = lane; j < count; j += kWave)
            out[j] = id0 + (int32_t)places[j];
        __builtin_amdgcn_wave_barrier();
        i = i_next;
        step = step_next;
        word = word_next;
        pre = pre_next;
    }
}

constexpr int kEmitThreads = 256;
__global__ __launch_bounds__(kEmitThreads) void rg_emit_kernel(RangeArgs a, int32_t *__restrict__ col_vertex)
{
    __shared__ uint16_t places[kEmitThreads / kWave][kEmitQuads * 128];
    const uint32_t wave = scalar(threadIdx.x / kWave);
    emit_steps(a, col_vertex, places[wave], blockIdx.x * (kEmitThreads / kWave) + wave, gridDim.x * (kEmitThreads / kWave));
}

static_assert((kMostGatheredMb + 1) * sizeof(int64_t) <= kRgWaves * kEmitQuads * 128 * sizeof(uint16_t), "minibatches out of step");
// Few entries: the first `emitters` workgroups emit, the others look entries up one by one.
__global__ __launch_bounds__(kRgThreads) void rg_emit_gather_kernel(RangeArgs a, int32_t *__restrict__ col_vertex, int emitters)
{
    __shared__ uint16_t places[kRgWaves][kEmitQuads * 128];
    if ((int)blockIdx.x < emitters) {
        const uint32_t wave = scalar(threadIdx.x / kWave);
        emit_steps(a, col_vertex, places[wave], blockIdx.x * kRgWaves + wave, (uint32_t)emitters * kRgWaves);
        return;
    }
    const int64_t x = (int64_t)blockIdx.x - emitters, nx = (int64_t)gridDim.x - emitters;
    auto column = [&](int64_t i, uint32_t id) -> int32_t {
        if ((int64_t)id >= a.n)
            return 0; // a seed outside [0, n), reported by the seed check
        const int64_t q = i * a.stride + (id >> 7);
        const uint4 v = a.bits[q];
        const uint32_t w = (id >> 5) & 3u, below = (1u << (id & 31u)) - 1u;
        const uint32_t word = w == 0 ? v.x : w == 1 ? v.y : w == 2 ? v.z : v.w;
        const int64_t r = range_of(a, id >> 7);
        return (int32_t)(a.first[i * a.H + r] - a.first[i * a.H]) +
               (int32_t)(a.pre[q] + (w > 0 ? __popc(v.x) : 0) + (w > 1 ? __popc(v.y) : 0) + (w > 2 ? __popc(v.z) : 0) + __popc(word & below));
    };
    // the entries (then the rows) of all minibatches one after the other, whose minibatch is found in LDS
    int64_t *begin = reinterpret_cast<int64_t *>(places); // k + 1 <= kMostGatheredMb
    for (int32_t i = threadIdx.x; i <= a.k; i += kRgThreads)
        begin[i] = a.rowptr[a.mb_rowoff[i]];
    __syncthreads();
    for (int64_t e = begin[0] + x * kRgThreads + threadIdx.x; e < begin[a.k]; e += nx * kRgThreads)
        a.col[e] = column(locate_segment(begin, a.k, e), (uint32_t)a.col[e]);
    if (!a.row_self)
        return;
    __syncthreads();
    for (int32_t i = threadIdx.x; i <= a.k; i += kRgThreads)
        begin[i] = a.mb_rowoff[i];
    __syncthreads();
    for (int64_t r = begin[0] + x * kRgThreads + threadIdx.x; r < begin[a.k]; r += nx * kRgThreads)
        a.row_self[r] = column(locate_segment(begin, a.k, r), (uint32_t)a.row_vertex[r]);
}

// Chunks of PER * 1024 entries of a minibatch (and, with row_self, of its rows behind them), in registers; `chunks`
// workgroups share a minibatch.  An id that has become a local column has bit 31 set until it is written.
constexpr uint32_t kFound = 0x80000000u;
// p[byte offset]: 32-bit offsets from addresses that are the same in all lanes keep the lanes' registers free
template <class T>
__device__ __forceinline__ const T *at_byte(const T *p, uint32_t byte)
{
    return reinterpret_cast<const T *>(reinterpret_cast<const char *>(p) + byte);
}
template <class T>
__device__ __forceinline__ T *at_byte(T *p, uint32_t byte)
{
    return reinterpret_cast<T *>(reinterpret_cast<char *>(p) + byte);
}
template <int PER>
__global__ __launch_bounds__(kRgThreads) void rg_lookup_kernel(RangeArgs a, int32_t chunks, int32_t passes, int32_t tq)
{
    extern __shared__ uint4 table4[]; // tq quads: per word (bits, columns of the minibatch before it), two words in 16 bytes
    const uint2 *table = reinterpret_cast<const uint2 *>(table4);
    const int tid = threadIdx.x;
    int i;
    uint32_t x0; // the first chunk of this workgroup
    die_order(blockIdx.x, (uint32_t)a.k, (uint32_t)chunks, i, x0);
    const int64_t r0 = a.mb_rowoff[i], r1 = a.mb_rowoff[i + 1];
    const int64_t e0 = a.rowptr[r0], e1 = a.rowptr[r1];
    const int64_t step = (int64_t)PER * kRgThreads;
    const int64_t entry_chunks = (e1 - e0 + step - 1) / step;
    const int64_t all_chunks = entry_chunks + (a.row_self ? (r1 - r0 + step - 1) / step : 0);
    const int64_t *__restrict__ first_i = a.first + (int64_t)i * a.H;
    const uint4 *__restrict__ bits_i = a.bits + (int64_t)i * a.stride;
    const uint32_t *__restrict__ pre_i = a.pre + (int64_t)i * a.stride;
    const int64_t first0 = first_i[0];
    const uint32_t quads = (uint32_t)a.quads;
    for (int64_t c = x0; c < all_chunks; c += chunks) {
        const bool entries = c < entry_chunks;
        const int64_t j0 = entries ? e0 + c * step : r0 + (c - entry_chunks) * step;
        const int32_t left = (int32_t)min<int64_t>(step, (entries ? e1 : r1) - j0);
        const int32_t *src = (entries ? (const int32_t *)a.col : a.row_vertex) + j0;
        // buffer accesses check the chunk's end themselves; offsets from a lane number that the compiler takes for a new one
        // each time are computed where they are used, not kept in 2 PER registers
        uint32_t lane4 = (uint32_t)tid * 4u;
        asm volatile("" : "+v"(lane4));
        const auto from = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(src), 0, left * 4, 0x00027000);
        uint32_t id[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q)
            id[q] = __builtin_amdgcn_raw_buffer_load_b32(from, (int)(lane4 + q * kRgThreads * 4u), 0, 0);
        uint4 bits[kTablePer];
        uint32_t pre[kTablePer];
        auto fetch = [&](int p) {
            uint32_t lane = (uint32_t)tid;
            asm volatile("" : "+v"(lane));
#pragma unroll
            for (int t = 0; t < kTablePer; ++t) {
                const uint32_t q = min((uint32_t)(p * tq) + min(t * kRgThreads + lane, (uint32_t)tq - 1u), quads - 1u); // (unused ones read the last)
                bits[t] = *at_byte(bits_i, q * 16u);
                pre[t] = *at_byte(pre_i, q * 4u) + (uint32_t)(*at_byte(first_i, range_of(a, q) * 8u) - first0);
            }
        };
        fetch(0);
#pragma unroll 1
        for (int p = 0; p < passes; ++p) {
            __syncthreads(); // the table of the pass before is done with
#pragma unroll
            for (int t = 0; t < kTablePer; ++t) {
                const int x = t * kRgThreads + tid;
                if (x < tq) {
                    const uint32_t p1 = pre[t] + __popc(bits[t].x), p2 = p1 + __popc(bits[t].y), p3 = p2 + __popc(bits[t].z);
                    table4[2 * x] = make_uint4(bits[t].x, pre[t], bits[t].y, p1);
                    table4[2 * x + 1] = make_uint4(bits[t].z, p2, bits[t].w, p3);
                }
            }
            __syncthreads();
            if (p + 1 < passes)
                fetch(p + 1);
            const uint32_t lo = (uint32_t)p * (uint32_t)tq * 128u;
            const uint32_t ids = (uint32_t)min((int64_t)tq * 128, a.n - (int64_t)lo);
            // eight reads in flight; an id outside the range reads the first word, as all of them do, and stays as it is
#pragma unroll
            for (int q0 = 0; q0 < PER; q0 += 8) {
                uint2 word[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const uint32_t rel = id[q0 + u] - lo;
                    word[u] = table[rel < ids ? rel >> 5 : 0u];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const uint32_t rel = id[q0 + u] - lo;
                    const uint32_t column = (word[u].y + __popc(word[u].x & ((1u << (rel & 31u)) - 1u))) | kFound;
                    id[q0 + u] = rel < ids ? column : id[q0 + u];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        asm volatile("" : "+v"(lane4));
        const auto to = __builtin_amdgcn_make_buffer_rsrc((entries ? a.col : a.row_self) + j0, 0, left * 4, 0x00027000);
#pragma unroll
        for (int q = 0; q < PER; ++q)
            __builtin_amdgcn_raw_buffer_store_b32(id[q] & ~kFound, to, (int)(lane4 + q * kRgThreads * 4u), 0, 0);
    }
}

static int64_t mark_ranges(int64_t n) { return ((n + 127) / 128 + kMarkQuads - 1) / kMarkQuads; }

// Measured on 0.1 to 0.6 million entries per minibatch and 2.4 million vertices, one workgroup per compute unit: a mark
// workgroup that counts takes 10 us and 76 ps per entry, one that does not 5 us and 150 ps (its range is wider: more ids set
// bits), the merging count 10 us and 4 TB/s.  Both run in whole rounds of the chip.
// most_bytes: of all bitmaps and counts together.
void plan_ranges(RangeArgs &a, int num_cu, double per_mb, int64_t most_bytes)
{
    double least = 0.0;
    for (int its = 1; its <= kMarkIts; ++its) {
        const int64_t H = (a.quads + its * kRgThreads - 1) / (its * kRgThreads);
        const double cost = (double)((a.k * H + num_cu - 1) / num_cu) * (per_mb * 76e-6 + 8.0 + 0.35 * its);
        if (its == 1 || cost < least) {
            least = cost;
            a.qw = its * kRgThreads;
            a.parts = 1;
        }
    }
    const int64_t stride = (a.quads + kRangeQuads - 1) / kRangeQuads * kRangeQuads;
    for (int32_t parts = 2; parts <= kMostParts && a.k * stride * (parts * 16 + 4) <= most_bytes; parts *= 2) {
        const double rounds = (double)((a.k * mark_ranges(a.n) * parts + num_cu - 1) / num_cu);
        const double cost = rounds * (per_mb / parts * 150e-6 + 5.0) + 10.0 + (double)a.k * parts * (double)a.n / 8 / 4e6;
        if (cost < least) {
            least = cost;
            a.qw = kRangeQuads;
            a.parts = parts;
        }
    }
}

int launch_ranges_mark(const Launch &L, const RangeArgs &a)
{
    static bool attr_set = false;
    if (!attr_set) {
        for (auto *kernel : {rg_mark_kernel<true>, rg_mark_kernel<false>})
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    kMarkQuads * (int)sizeof(uint4)) != hipSuccess)
                (void)hipGetLastError(); // not required on every runtime; the launch below reports real failures
        attr_set = true;
    }
    if (a.parts == 1) {
        hipLaunchKernelGGL(rg_mark_kernel<true>, dim3((unsigned)(a.k * a.H)), dim3(kRgThreads), (size_t)a.qw * sizeof(uint4), L.stream, a, a.qw);
    } else {
        const int64_t H = mark_ranges(a.n);
        const int32_t mq = (int32_t)((a.quads + H - 1) / H);
        hipLaunchKernelGGL(rg_mark_kernel<false>, dim3((unsigned)(a.k * H * a.parts)), dim3(kRgThreads), (size_t)mq * sizeof(uint4), L.stream, a, mq);
        hipLaunchKernelGGL(rg_count_kernel, dim3((unsigned)(a.k * a.H)), dim3(kRgThreads), 0, L.stream, a);
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

void launch_ranges_count(const Launch &L, const RangeArgs &a)
{
    hipLaunchKernelGGL(rg_count_kernel, dim3((unsigned)(a.k * a.H)), dim3(kRgThreads), 0, L.stream, a);
}

void launch_ranges_emit(const Launch &L, const RangeArgs &a, int32_t *col_vertex)
{
    const int64_t steps = (int64_t)a.k * ((a.quads + kEmitQuads - 1) / kEmitQuads);
    const int64_t waves = kEmitThreads / kWave;
    hipLaunchKernelGGL(rg_emit_kernel, dim3(grid_for(L, (steps + waves - 1) / waves, 8)), dim3(kEmitThreads), 0, L.stream, a, col_vertex);
}

void launch_ranges_emit_gather(const Launch &L, const RangeArgs &a, int32_t *col_vertex, int64_t entries)
{
    const int64_t steps = (int64_t)a.k * ((a.quads + kEmitQuads - 1) / kEmitQuads);
    const int emitters = grid_for(L, (steps + kRgWaves - 1) / kRgWaves, 1), gatherers = grid_for(L, entries / kRgThreads + 1, 1);
    hipLaunchKernelGGL(rg_emit_gather_kernel, dim3(emitters + gatherers), dim3(kRgThreads), 0, L.stream, a, col_vertex, emitters);
}

int ranges_passes(int64_t n) { return (int)(((n + 127) / 128 + kTableQuads - 1) / kTableQuads); }

int launch_ranges_lookup(const Launch &L, const RangeArgs &a, double per_mb)
{
    void (*const kernels[4])(RangeArgs, int32_t, int32_t, int32_t) = {rg_lookup_kernel<8>, rg_lookup_kernel<16>, rg_lookup_kernel<32>,
                                                                      rg_lookup_kernel<56>}; // (64 do not fit the registers)
    static bool attr_set = false;
    if (!attr_set) {
        for (auto *kernel : kernels)
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    kTableQuads * 2 * (int)sizeof(uint4)) != hipSuccess)
                (void)hipGetLastError();
        attr_set = true;
    }
    const int passes = ranges_passes(a.n);
    const int tq = (int)((a.quads + passes - 1) / passes);
    // the chunk length that takes least: whole rounds of one workgroup per compute unit, each of them `passes` tables (1.8 us)
    // and look-ups (0.06 us per entry of a thread)
    constexpr int pers[4] = {8, 16, 32, 56};
    int best = 0;
    int32_t best_chunks = 1;
    double least = 0.0;
    for (int x = 0; x < 4; ++x) {
        const int per = pers[x];
        const int32_t chunks = std::max(1, (int32_t)(per_mb * 1.01 / (per * kRgThreads) + 0.999));
        const double rounds = (double)(((int64_t)a.k * chunks + L.num_cu - 1) / L.num_cu);
        const double cost = rounds * passes * (1.8 + 0.06 * per);
        if (x == 0 || cost < least) {
            least = cost;
            best = x;
            best_chunks = chunks;
        }
    }
    hipLaunchKernelGGL(kernels[best], dim3((unsigned)((int64_t)a.k * best_chunks)), dim3(kRgThreads), (size_t)tq * 2 * sizeof(uint4),
                       L.stream, a, best_chunks, passes, tq);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

} // namespace bms
