// Layer-wise (LADIES) bulk sampling, Sec. 4.2 of arxiv 2311.02909: the path that accumulates the
// column counts of P = Q A in LDS.
//
// The rows of A are sorted by column, so the neighbours of a frontier row that fall into a window
// of 2^16 vertex ids form one contiguous piece of its adjacency list.  One hop, all k minibatches:
//   ldw_rows        extents of the frontier's rows, exclusive scan of their degrees = the gathered order; in the first hop
//                   the frontier is the seeds, which are checked and copied beside it
//   ldw_plan, ldw_tile_rows
//                   the gathered order (the neighbour lists of the stacked frontier laid end to end) cut into
//                   tiles of 1024..4096 positions (few gathered neighbours: small tiles, so that every wave still
//                   gets some) that never straddle minibatches; the row each tile starts in
//   ldw_bounds      where every row crosses every window boundary (lower bounds, one list per row).  A row's list
//                   depends on its vertex alone: when the lists of all n vertices fit in memory they are computed
//                   once per graph (one wave per tile streams its pieces of rows, the "hop" being the whole
//                   graph) and a hop only copies the lists of its rows; else the hop streams its rows for them.
//                   Either way the lists are turned window-major for the next kernel.  With the index and k < 1024 there
//                   are none of these launches: further workgroups of ldw_rows copy the lists, further ones of
//                   ldw_p_place or ldw_win_scan make the plan and find the tile rows, which the extraction needs first
//   ldw_accumulate  one workgroup per (minibatch, window): 2^16 packed counters of 16 bits (128 KB) or 8 bits in LDS;
//                   every row's piece of the window adds 1 per neighbour (e_v cannot exceed the number of frontier
//                   rows, which this path keeps below 2^16); the waves then take its sixteenths
//                   (parts) out: the nonzero counters leave in ascending column order as 4-byte entries
//                   (column - window start, e_v), or as a bit per column and a byte per entry, into room claimed from a
//                   device-wide cursor; columns and weight of every part and window are recorded
//   ldw_p_place     the parts copied to their place in P; inclusive prefix sums of the integer weights (e_v or e_v^2) on
//                   the way, one kept per 16 entries (NORM stays implicit: draws are integers below the row sum).  A
//                   workgroup takes a pair and adds up the sizes of those before it
//   ldw_win_scan, ldw_p_copy
//                   the same of more than 2048 pairs: the places by a launch of their own, a wave per part
//   ldw_draw        SAMPLE (Sec. 4.2.2): one workgroup per minibatch, or several with a share of the draws each: s draws, each the smallest t
//                   with prefix[t] > r, sorted in LDS, duplicates dropped -> sampled columns, at their place in the stack
//   ldw_extract     EXTRACT (Sec. 4.2.3): the sampled columns of the minibatch sit in an LDS hash
//                   table (column -> local index); one wave per tile streams the gathered order a
//                   second time and keeps the neighbours found in the table ((Q_R A) Q_C), in
//                   row order, piece by piece; rows are then sized by a scan and their pieces
//                   copied to their place (ldw_extract_place)
// A launch costs about 5 us on the device however little it does, and most of these do little: where a kernel needs sums over
// its own workgroups (rows, minibatches), the workgroups add up those before them (sum_before) instead of leaving it to a
// kernel in between.  32 x 512 seeds, 3 x 512 samples, 2.4 M vertices: 18 -> 6 launches a hop.
// A call that sizes its buffers from an earlier call of the same shape runs all of these behind LwHop::giveup.
#include "bms_device.h"
#include "bms_internal.h"
#include "publish.h"
#include <algorithm>

namespace bms {

constexpr int kWinIds = 1 << kWinShift;
constexpr int kPartIds = kWinIds / kWinParts; // a part of a window
constexpr int kWaveWords = 2048;         // counter words that a wave of the accumulation takes out: a part in 16 bits, two in 8
constexpr uint32_t kEmptySlot = 0xFFFFFFFFu;
constexpr int kExtThreads = 1024; // the waves of a workgroup share one hash table
constexpr int kExtWaves = kExtThreads / kWave;
constexpr int kAccUnroll = 8;              // 16-byte loads per lane and span
constexpr int kAccChunks = kWave * kAccUnroll; // aligned 16-byte chunks per span: one per lane and load
constexpr int kAccFlush = 4;               // entries per lane on their way out at a time
constexpr int kAccListed = 956;            // counters in use that a wave lists in LDS at a time
struct AccPiece {                          // one nonempty piece of a wave's rows
    int64_t origin;                        // byte address of its first chunk - 16 * chunks of the batch before it
    int32_t lo, hi;                        // its first entry and the one behind its last, counted from origin
};
struct AccWave {
    union { // in turn
        AccPiece piece[kWave];     // one record per nonempty piece of a batch, by rank
        alignas(8) uint16_t list[kAccListed + 4]; // (entries that leave four to a word: up to three behind the listing before)
    };
    uint32_t starts[2 * kAccUnroll]; // a bit per chunk of a span: a piece starts there
};
// A workgroup of the accumulation: 16 waves with counters of 16 bits (a compute unit holds one), or 8 with counters of 8 bits
// (it holds two).
template <bool NARROW>
constexpr int kAccThreads = NARROW ? 512 : 1024;
template <bool NARROW>
struct AccShared {
    static constexpr int kWaves = kAccThreads<NARROW> / kWave;
    AccWave wave[kWaves];
    unsigned long long claimed; // where the pair's entries start in the staging array
    unsigned long long weight;  // of the pair's columns
    uint32_t cnt[kWinParts];    // columns in the parts
    uint32_t missing[kWaves];   // with 8 bits: neighbours in the wave's rows - those that its counters show
};
template <bool NARROW>
struct AccLds {
    alignas(16) uint32_t cnt[AccShared<NARROW>::kWaves * kWaveWords]; // packed counters
    AccShared<NARROW> sh;
};
static_assert(sizeof(AccLds<false>) <= 160 * 1024 && 2 * sizeof(AccLds<true>) <= 160 * 1024, "does not fit a compute unit");
// A part is staged in one of two forms (part_base: 2 x its first word in tmp_ent, + 1 with masks):
//   entries  a word each, (column - the window's first id) << 16 | e_v
//   masks    a bit per column of the part in use, then a byte per entry: e_v.  Only of counters of 8 bits, and of parts with at
//            least kMaskFrom columns, where it is the shorter one (so that what holds the entries holds either form)
constexpr uint32_t kMaskWords = kPartIds / 32;
constexpr uint32_t kMaskFrom = 256;
static_assert(kMaskWords + (kMaskFrom + 3) / 4 <= kMaskFrom, "not the shorter one");
constexpr int64_t kMaskEntries = 256; // of a part on average, from which on (launch_ldw_accumulate)
__device__ inline uint32_t staged_words(uint32_t columns, bool as_masks)
{
    return as_masks && columns >= kMaskFrom ? kMaskWords + (columns + 3u) / 4u : columns;
}
using FourPlaces = uint64_t __attribute__((may_alias));
using I32x2_a4 = int32_t __attribute__((ext_vector_type(2), aligned(4)));
using U32x4_a4 = uint32_t __attribute__((ext_vector_type(4), aligned(4)));
using U32x2_a4 = uint32_t __attribute__((ext_vector_type(2), aligned(4)));

constexpr int kPrefixBlock = 16; // entries of P per kept prefix sum
constexpr int kStreamUnroll = 8; // neighbours per lane in flight in the two streaming passes
constexpr int kDrawTop = 2048;                    // recorded weight sums of P that a drawing workgroup keeps in LDS

__device__ inline uint64_t ldw_weight(uint32_t cnt, int squared)
{
    return squared ? (uint64_t)cnt * (uint64_t)cnt : (uint64_t)cnt;
}

// ---------------------------------------------------------------------------------------------
// Rows: extents, the gathered order (exclusive scan of the degrees), 256 rows per workgroup
// ---------------------------------------------------------------------------------------------
__device__ inline void transpose_bounds(const LwHop &a, const int32_t *row_vertex, int64_t nrows, uint32_t *room, int64_t x, int64_t nx);

// The first `tiles` workgroups take the rows.  With the index, workgroups behind them turn the rows' lists window-major for the
// accumulation (a launch of its own before, 6 us of every hop; both only need the frontier).  In the first hop (a.seeds) the frontier
// is the seeds themselves, and k workgroups in between check those of a minibatch each, copy them and leave where it begins (a launch
// before, 4 us of every call): nobody in this launch reads what they write.
__global__ __launch_bounds__(kLwRows) void ldw_rows_kernel(LwHop a, Lookback lb, int64_t *gathered_out, int tiles)
{
    extern __shared__ uint32_t rows_lds[]; // hash table of the seeds, or room for transpose_bounds
    __shared__ int64_t smem[kLwRows / kWave];
    __shared__ uint32_t number_s;
    const int tid = threadIdx.x;
    const int32_t *row_vertex = a.seeds ? a.seeds : a.row_vertex;
    if ((int)blockIdx.x >= tiles) {
        const int checks = a.seeds ? a.k : 0, x = (int)blockIdx.x - tiles;
        if (x < checks) {
            if (tid == 0) {
                a.seed_rowoff[x] = (int64_t)x * a.b;
                if (x == a.k - 1)
                    a.seed_rowoff[a.k] = (int64_t)a.k * a.b;
            }
            check_seeds<kLwRows>(a.seeds, x, a.b, a.n, a.seed_slots, a.seed_shift, rows_lds, a.seed_copy, a.seed_flags);
        } else {
            const int64_t nrows = a.seeds ? (int64_t)a.k * a.b : uniform_load(a.mb_rowoff + a.k);
            transpose_bounds(a, row_vertex, nrows, rows_lds, x - checks, (int64_t)gridDim.x - tiles - checks);
        }
        return;
    }
    const uint32_t t = scalar(take_number(lb, &number_s));
    const int64_t R = a.seeds ? (int64_t)a.k * a.b : uniform_load(a.mb_rowoff + a.k);
    const int64_t r0 = (int64_t)t * kLwRows, r = r0 + tid;
    if (t > 0 && r0 >= R)
        return; // nobody with rows comes after
    const int32_t v = r < R ? row_vertex[r] : -1;
    // the minibatch of the first row, while the vertices are on their way; mostly that of all rows
    int lo = 0;
    if (!a.seeds)
        for (int hi = a.k; hi - lo > 1;) {
            const int mid = (lo + hi) >> 1;
            if (uniform_load(a.mb_rowoff + mid) <= r0)
                lo = mid;
            else
                hi = mid;
        }
    int64x2_a8 extent = {0, 0};
    if (v >= 0 && (int64_t)v < a.n)
        extent = row_extent(a.A_rowptr, v);
    int mb = lo;
    if (a.seeds)
        mb = (int)((uint32_t)r / (uint32_t)a.b); // fewer than 2^18 rows
    else if (uniform_load(a.mb_rowoff + lo + 1) < min(r0 + kLwRows, R) && r < R)
        mb = locate_segment(a.mb_rowoff, a.k, r);
    const int64_t beg = extent[0], deg = extent[1] - extent[0];
    int64_t total;
    const int64_t ex = block_exclusive_scan<int64_t, kLwRows>(deg, smem, total);
    const int64_t before = sum_before<kLwRows>(lb, t, total, smem);
    if (r < R) {
        a.row_beg[r] = beg;
        a.gather_off[r] = before + ex;
        a.row_mb[r] = mb;
        a.out_rowptr[r] = 0; // per-row counters of the extraction pass
    }
    if ((int64_t)(t + 1) * kLwRows < R)
        return;
    const int64_t all = before + total;
    const bool too_many = a.giveup && all > a.gathered_cap; // the kernels after this one see it
    if (tid == 0) {
        a.gather_off[R] = all;
        a.out_rowptr[R] = 0;
    }
    if (a.seeds) { // the call's scalars start anew, the staging cursor among them
        if (tid < 64) {
            int64_t *slot = a.scalars + tid;
            *slot = slot == gathered_out ? all : (too_many && slot == reinterpret_cast<int64_t *>(a.giveup)) ? 1 : 0;
        }
    } else if (tid == 0) {
        *gathered_out = all;
        *a.cursor = 0;
        if (too_many)
            *a.giveup = 1;
    }
}

// ---------------------------------------------------------------------------------------------
// Tiles of the gathered order
// ---------------------------------------------------------------------------------------------
// One workgroup: where each minibatch starts in the gathered order (mb_goff), the tiles before each minibatch
// (mb_gtileoff); the tile counters of the extraction and the staging cursor of the accumulation start at zero.
__global__ __launch_bounds__(1024) void ldw_plan_kernel(LwHop a)
{
    __shared__ int64_t smem[16];
    __shared__ int64_t carry_s;
    if (threadIdx.x == 0) {
        carry_s = 0;
        if (a.cursor)
            *a.cursor = 0;
        if (a.giveup && a.gather_off[a.mb_rowoff[a.k]] > a.gathered_cap)
            *a.giveup = 1; // the kernels after this one see it: they are launched after this one ends
    }
    __syncthreads();
    for (int32_t base = 0; base <= a.k; base += 1024) {
        const int32_t i = base + threadIdx.x;
        int64_t cnt = 0;
        if (i <= a.k) {
            const int64_t g0 = a.gather_off[a.mb_rowoff[i]];
            a.mb_goff[i] = g0;
            if (a.tile_queue)
                a.tile_queue[i * kQueueStride] = 0;
            if (i < a.k)
                cnt = (a.gather_off[a.mb_rowoff[i + 1]] - g0 + a.tile - 1) / a.tile;
        }
        int64_t total;
        const int64_t ex = block_exclusive_scan<int64_t, 1024>(cnt, smem, total);
        const int64_t carry = carry_s;
        if (i <= a.k)
            a.mb_gtileoff[i] = carry + ex; // entry k: all tiles
        __syncthreads();
        if (threadIdx.x == 0)
            carry_s = carry + total;
        __syncthreads();
    }
}

// tile_row[x] = the row that holds the first position of tile x (the last row starting at or before it)
__global__ __launch_bounds__(256) void ldw_tile_rows_kernel(LwHop a)
{
    if (a.giveup && *a.giveup)
        return;
    const int64_t ntiles = a.mb_gtileoff[a.k];
    for (int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x; x < ntiles; x += (int64_t)gridDim.x * 256) {
        const int i = locate_segment(a.mb_gtileoff, a.k, x);
        const int64_t g0 = a.mb_goff[i] + (x - a.mb_gtileoff[i]) * a.tile;
        int64_t lo = a.mb_rowoff[i], hi = a.mb_rowoff[i + 1];
        while (hi - lo > 1) {
            const int64_t mid = (lo + hi) >> 1;
            if (a.gather_off[mid] <= g0)
                lo = mid;
            else
                hi = mid;
        }
        a.tile_row[x] = lo;
    }
}

// Walks the pieces of rows inside tile [g0, g1) of the gathered order, starting in row r0 (the row that holds
// g0), and calls body(r, rs, re, shift, g, pe) for each: row r spans gathered positions [rs, re), the piece is
// [g, pe), and A_col[shift + p] is the neighbour at position p.  The extent of the following row is fetched
// while a piece is being worked on, so a new piece does not start with a chain of dependent loads.
template <class Body>
__device__ inline void ldw_walk_tile(const LwHop &a, int64_t g0, int64_t g1, int64_t r0, int64_t nrows, Body body)
{
    int64_t g = g0, r = r0;
    int64_t rs = a.gather_off[r], re = a.gather_off[r + 1], beg = a.row_beg[r];
    while (g < g1) {
        const int64_t rn = r + 1 < nrows ? r + 1 : r;
        const int64_t next_re = a.gather_off[rn + 1], next_beg = a.row_beg[rn];
        const int64_t pe = min(re, g1);
        body(r, rs, re, beg - rs, g, pe);
        g = pe;
        if (pe == re) {
            ++r;
            rs = re;
            re = next_re;
            beg = next_beg;
            while (re <= g && g < g1) { // rows without neighbours
                ++r;
                rs = re;
                re = a.gather_off[r + 1];
                beg = a.row_beg[r];
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// bounds[r * (nwin + 1) + w] = number of neighbours of row r with id < w * 2^16, w = 0..nwin (row-major:
// the wave that streams a row writes its boundaries next to each other)
// (rows without neighbours are skipped: their entries are never read)
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void ldw_bounds_kernel(LwHop a)
{
    if (a.giveup && *a.giveup)
        return;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t ntiles = a.mb_gtileoff[a.k];
    const int64_t nrows = a.mb_rowoff[a.k];
    for (int64_t x = (int64_t)blockIdx.x * 4 + threadIdx.x / kWave; x < ntiles; x += (int64_t)gridDim.x * 4) {
        const int i = locate_segment(a.mb_gtileoff, a.k, x);
        const int64_t g0 = a.mb_goff[i] + (x - a.mb_gtileoff[i]) * a.tile;
        const int64_t g1 = min(g0 + a.tile, a.mb_goff[i + 1]);
        ldw_walk_tile(a, g0, g1, a.tile_row[x], nrows,
                      [&](int64_t r, int64_t rs, int64_t re, int64_t shift, int64_t g, int64_t pe) {
            uint32_t *__restrict__ out = a.bounds + r * (a.nwin + 1);
            // when the row ends inside the tile, position `re` acts as one more entry that lies in
            // window nwin: it closes every window left
            const int64_t last = pe == re ? pe : pe - 1;
            int32_t carry = g == rs ? -1 : (a.A_col[shift + g - 1] >> kWinShift); // window of the entry before
            for (int64_t p0 = g; p0 <= last; p0 += kStreamUnroll * kWave) {
                // 32-bit slot numbers from here on: slot x of the step is gathered position p0 + x
                const int32_t *__restrict__ from = a.A_col + (shift + p0);
                const int32_t nreal = (int32_t)min<int64_t>(re - p0, kStreamUnroll * kWave); // slots that hold a neighbour
                const int32_t xlast = (int32_t)min<int64_t>(last - p0, kStreamUnroll * kWave - 1);
                const uint32_t pos0 = (uint32_t)(p0 - rs);
                int32_t wv[kStreamUnroll];
#pragma unroll
                for (int u = 0; u < kStreamUnroll; ++u) {
                    const int32_t x = u * kWave + lane;
                    wv[u] = x < nreal && x <= xlast ? (from[x] >> kWinShift) : a.nwin;
                }
#pragma unroll
                for (int u = 0; u < kStreamUnroll; ++u) {
                    const int32_t x = u * kWave + lane;
                    // window of the entry one lane below (lane 0: of the entry before the step): a lane shift in
                    // the vector unit, not a trip through LDS
                    const int32_t pw = __builtin_amdgcn_update_dpp(carry, wv[u], 0x138 /* wave_shr:1 */, 0xF, 0xF, false);
                    if (x <= xlast) // this entry is the first at or past the boundaries pw+1 .. wv
                        for (int32_t w = pw + 1; w <= wv[u]; ++w)
                            out[w] = pos0 + (uint32_t)x;
                    carry = __builtin_amdgcn_readlane(wv[u], kWave - 1);
                }
            }
        });
    }
}

// The boundary lists turned window-major (bounds_t[w * rows_bound + r]): the accumulation reads one window of
// all rows at a time.  The list of row r comes from this hop's boundary pass, or, when the graph carries an index of every vertex's
// list, from the index entry of the row's vertex (all zeros for vertices without neighbours, and so here for their rows).  64 rows and
// a.bounds_width boundaries at a time through LDS, both sides coalesced: a list is read as few pieces of equal width, its words dealt to the
// lanes in their order.  room: BoundsPieces::lds bytes of LDS.  256 threads, workgroup x of nx.
// Three layers of 64 x 1024 seeds, 133 windows: the launch 154 -> 130 us, in squares of 64 x 64 before, whose last ones had 6 of 64
// words and which read the lists' lines twice; 32 x 512, 38 windows: 38 -> 33.
constexpr int kBoundsRows = 64;
struct BoundsPieces {
    int32_t width;
    int64_t tiles;
    size_t lds;
};
// Pieces of up to 64 boundaries are one trip to memory for a thread's 16 reads, those of up to 128 are two, with the lists' lines cut
// less often.  The trip counts as long as the chip holds all of the pieces at a time (four workgroups per compute unit).  Two layers, the launches by
// 128 and by 64: 8 x 64 seeds, 134 boundaries 16.4 and 12.2 us, 1695 20.6 and 14.6; 32 x 512, 81 19.4 and 16.0, 224 22.6 and 19.2; 64 x 1024,
// 81 39.4 and 41.6, 224 51.3 and 55.0; 64 x 512, 1695 170 and 180.
static BoundsPieces bounds_pieces(const Launch &L, const LwHop &a)
{
    const int64_t ncols = (int64_t)a.nwin + 1, row_tiles = (a.rows_bound + kBoundsRows - 1) / kBoundsRows;
    const int64_t most = row_tiles * ((ncols + 63) / 64) <= (int64_t)L.num_cu * 4 ? 64 : 128;
    const int64_t pieces = (ncols + most - 1) / most, width = (ncols + pieces - 1) / pieces;
    // (rows of an odd number of words: their words at one place are in different banks)
    return {(int32_t)width, pieces * row_tiles, (kBoundsRows * (size_t)(width | 1) + kBoundsRows) * sizeof(uint32_t)};
}
__device__ inline void transpose_bounds(const LwHop &a, const int32_t *row_vertex, int64_t nrows, uint32_t *room, int64_t x, int64_t nx)
{
    constexpr int NT = 256, kEach = 16; // reads in flight per thread
    const uint32_t ncols = (uint32_t)a.nwin + 1u, width = (uint32_t)a.bounds_width, pieces = (ncols + width - 1) / width;
    const uint32_t stride = width | 1u;
    int32_t *list_of = reinterpret_cast<int32_t *>(room + kBoundsRows * stride); // whose list a row has; -1: none
    const int64_t tiles = (int64_t)pieces * ((nrows + kBoundsRows - 1) / kBoundsRows);
    const uint32_t *lists = a.index ? a.index : a.bounds;
    const int tid = threadIdx.x, tx = tid & 63, ty = tid >> 6;
    for (int64_t t = x; t < tiles; t += nx) {
        const int64_t r0 = t / pieces * kBoundsRows;
        const uint32_t c0 = (uint32_t)(t % pieces) * width, w = min(width, ncols - c0);
        if (tid < kBoundsRows) {
            const int64_t r = r0 + tid;
            int32_t of = -1;
            if (r < nrows && a.index) { // a seed outside [0, n) is an error reported elsewhere; its row has no neighbours
                const int32_t v = row_vertex[r];
                of = v >= 0 && (int64_t)v < a.n ? v : -1;
            } else if (r < nrows) { // (a row without neighbours has no boundaries on record)
                of = a.gather_off[r + 1] != a.gather_off[r] ? tid : -1;
            }
            list_of[tid] = of;
        }
        __syncthreads();
        const int64_t first = a.index ? 0 : r0; // list of number 0
        uint32_t row = (uint32_t)tid / w, col = (uint32_t)tid - row * w;
        const uint32_t row_step = NT / w, col_step = NT - row_step * w;
        while (row < (uint32_t)kBoundsRows) { // (of some threads: the others have no more)
            uint32_t y[kEach], place[kEach];
#pragma unroll
            for (int q = 0; q < kEach; ++q) {
                y[q] = 0;
                place[q] = row * stride + col;
                const int32_t of = row < (uint32_t)kBoundsRows ? list_of[row] : -1;
                if (of >= 0)
                    y[q] = lists[(first + of) * ncols + c0 + col];
                if (row >= (uint32_t)kBoundsRows)
                    place[q] = ~0u;
                row += row_step;
                col += col_step;
                if (col >= w) {
                    col -= w;
                    ++row;
                }
            }
#pragma unroll
            for (int q = 0; q < kEach; ++q)
                if (place[q] != ~0u)
                    room[place[q]] = y[q];
        }
        __syncthreads();
        for (uint32_t y = ty; y < w; y += NT / 64)
            if (r0 + tx < nrows)
                a.bounds_t[(int64_t)(c0 + y) * a.rows_bound + r0 + tx] = room[tx * stride + y];
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void ldw_bounds_transpose_kernel(LwHop a)
{
    extern __shared__ uint32_t bounds_lds[];
    if (a.giveup && *a.giveup)
        return;
    transpose_bounds(a, a.row_vertex, a.mb_rowoff[a.k], bounds_lds, blockIdx.x, gridDim.x);
}

// Plan and tile rows by workgroups of a launch that does something else as well (hops with the index, k < kPlanMb): planner x of
// nx makes the plan for itself (the first one leaves it for the kernels that follow) and then finds tile rows.  NT threads.
constexpr int kPlanMb = 1024;
struct PlanShared {
    int64_t goff[kPlanMb], tileoff[kPlanMb];
};
template <int NT>
__device__ inline void plan_tiles(const LwHop &a, PlanShared &p, int64_t *smem /* NT / 64 */, int x, int nx)
{
    const int tid = threadIdx.x;
    const bool first = x == 0;
    for (int32_t i = tid; i <= a.k; i += NT)
        p.goff[i] = a.gather_off[a.mb_rowoff[i]];
    __syncthreads();
    int64_t carry = 0;
    for (int32_t base = 0; base <= a.k; base += NT) {
        const int32_t i = base + tid;
        const int64_t cnt = i < a.k ? (p.goff[i + 1] - p.goff[i] + a.tile - 1) / a.tile : 0;
        int64_t total;
        const int64_t ex = carry + block_exclusive_scan<int64_t, NT>(cnt, smem, total);
        if (i <= a.k)
            p.tileoff[i] = ex; // entry k: all tiles
        carry += total;
    }
    __syncthreads();
    if (first)
        for (int32_t i = tid; i <= a.k; i += NT) {
            a.mb_goff[i] = p.goff[i];
            a.mb_gtileoff[i] = p.tileoff[i];
            a.tile_queue[i * kQueueStride] = 0;
        }
    // A row holds the first positions of the tiles that start inside it: mostly none or one, found without a search (9 steps
    // through memory per tile of 512 rows); a row that holds many is given to the whole wave.
    const int64_t R = uniform_load(a.mb_rowoff + a.k);
    const int shift = __ffs(a.tile) - 1, lane = tid & (kWave - 1);
    for (int64_t r0 = (int64_t)x * NT + (tid - lane); r0 < R; r0 += (int64_t)nx * NT) {
        const int64_t r = r0 + lane;
        int64_t from = 0, count = 0; // tiles
        if (r < R) {
            const int64_t begin = a.gather_off[r], end = a.gather_off[r + 1];
            const int i = a.row_mb[r];
            const int64_t y = (begin - p.goff[i] + a.tile - 1) >> shift;
            from = p.tileoff[i] + y;
            count = ((end - p.goff[i] + a.tile - 1) >> shift) - y;
        }
        for (uint64_t many = __ballot(count > 8); many; many &= many - 1ull) {
            const int owner = __ffsll((unsigned long long)many) - 1;
            const int64_t x0 = lane_value(from, owner), n = lane_value(count, owner);
            for (int64_t y = lane; y < n; y += kWave)
                a.tile_row[x0 + y] = r0 + owner;
        }
        if (count <= 8)
            for (int64_t y = 0; y < count; ++y)
                a.tile_row[from + y] = r;
    }
}

// ---------------------------------------------------------------------------------------------
// P = Q A, one (minibatch, window) pair per workgroup at a time
// ---------------------------------------------------------------------------------------------
// both 16-bit halves, each min(half, 1)
__device__ inline uint32_t at_most_one(uint32_t x)
{
    using Halves = uint16_t __attribute__((ext_vector_type(2)));
    union {
        uint32_t whole;
        Halves halves;
    } v{x};
    const Halves one = {1, 1};
    v.halves = __builtin_elementwise_min(v.halves, one);
    return v.whole;
}

// A compute unit's LDS holds one workgroup with counters of 16 bits, whose waves are all in the same phase, or two with counters of
// 8 bits (NARROW), which fill one another's waits:
//   gather   a pair's first span of chunks is asked for while the counters of the pair before it leave
//   count    64 consecutive counters per lane: a bit for each that is in use, columns and weight of the wave's parts.  8 bits: a
//            pair with a counter that passed 255 is found by the sum of all counters, and counted anew half by half in 16 bits
//   write    a lane lists its counters in use, in column order, in LDS; the entries leave 64 to a store, or their bytes 256 to a
//            store behind the bits of the count, into room claimed for exactly as many (the claim is on its way while the lists
//            are made).  The latter writes 0.46 instead of 0.97 GB in three layers of 64 x 1024 seeds (1.14 -> 1.05 ms)
// Bound by vector instructions (half of the time), LDS (a third) and the lines of the pieces, none of them alone.  Few rows lie in half
// waves, so that all waves have some.  Weights e_v and e_v^2 are kernels of their own: decided inside, at every word, the branch kept the
// LDS reads from overlapping.  The chunks are read from addresses that the compiler knows to be memory: read from just any, each LDS addition waited
// for the one before it.  64 x 1024 seeds, 2048 samples, 8.7 M vertices (27 k neighbours per pair), one hop: 650 us, 560 by that and
// the shorter instruction sequences, 472 by counters of 8 bits as well; 32 x 512 seeds, 512 samples, 2.4 M vertices: 45 -> 36.
// Tried and slower: two spans of fewer loads in flight (1.15 times on the former), the next pair's loads dealt out between the
// steps of the count (1.14), all 64 lanes adding, those without an entry nothing (1.04: an LDS addition costs by active lanes),
// P written here at its final place, found by looking back over the sizes of the pairs before (1.2 to 1.7 times accumulation
// and copy together: it ties all workgroups to the slowest one of every round).
template <bool SQUARED, bool NARROW, bool MASKS>
__device__ __forceinline__ void accumulate(const LwHop &a)
{
    __shared__ AccLds<NARROW> lds; // (at a place that the compiler knows: an addition less per neighbour)
    if (a.giveup && *a.giveup)
        return;
    constexpr int NT = kAccThreads<NARROW>, NW = NT / kWave;
    uint32_t *cnt = lds.cnt;
    AccShared<NARROW> &sh = lds.sh;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = (int)scalar((uint32_t)tid / kWave);
    AccWave &me = sh.wave[wave];
    const int64_t A0 = (int64_t)reinterpret_cast<uintptr_t>(a.A_col);
    const uint32_t nwin = (uint32_t)a.nwin, nblk = (uint32_t)a.k * nwin; // (at most 2^16 minibatches and 2^15 windows)
    for (int x = tid; x < NW * kWaveWords / 4; x += NT)
        reinterpret_cast<uint4 *>(cnt)[x] = make_uint4(0, 0, 0, 0);
    if (tid == 0)
        sh.weight = 0;
    __syncthreads();
    // Workgroups are handed to the chip's 8 dies in turn, and each die has its own last-level cache.  Within a
    // round of gridDim.x (minibatch, window) pairs, die x takes a run of consecutive windows, so the memory
    // lines that hold the end of one window's piece and the start of the next one's are fetched once.
    const uint32_t G = gridDim.x;
    auto pair_of = [&](uint32_t round) -> uint32_t { // of the workgroup; nblk: none (nor in later rounds)
        const uint32_t p = blockIdx.x, at = G % 8 == 0 ? (p % 8) * (G / 8) + p / 8 : p;
        const uint64_t blk = (uint64_t)round * G + at;
        return blk < nblk ? (uint32_t)blk : nblk;
    };
    // A batch: the wave's rows first .. first + rows - 1 of a pair's minibatch, rows <= 64.  With few rows all waves get some.
    uint32_t window = 0;             // of the pair
    int32_t first = 0, rows = 0, all = 0; // all: rows of the minibatch
    int64_t r0 = 0;                  // its first row
    // the piece of the batch's row of this lane: boundaries in the row, where the row begins (the values are looked at where
    // they are used: the loads have until then)
    uint32_t bound0 = 0, bound1 = 0;
    int64_t row_beg = 0;
    uint32_t have = 0;               // neighbours in the pieces of this lane
    uint32_t u0 = 0, total = 0, ustart = 0; // chunks of the batch: those asked for, all, before the lane's piece
    auto fetch_pieces = [&]() {
        bound0 = bound1 = 0;
        row_beg = 0;
        u0 = 0;
        if (lane < min(rows, all - first)) {
            const int64_t r = r0 + first;
            const uint32_t *__restrict__ lo_b = a.bounds_t + (int64_t)window * a.rows_bound + r; // boundary w of the rows
            bound0 = lo_b[lane];
            bound1 = lo_b[a.rows_bound + lane];
            row_beg = (a.row_beg + r)[lane];
        }
    };
    auto begin_pair = [&](uint32_t blk) {
        first = rows = all = 0;
        if (blk < nblk) {
            const uint32_t i = blk / nwin;
            window = blk - i * nwin;
            r0 = uniform_load(a.mb_rowoff + i);
            all = (int32_t)(uniform_load(a.mb_rowoff + i + 1) - r0);
            rows = all <= NW * (kWave / 2) ? kWave / 2 : kWave;
            first = wave * rows;
        }
        fetch_pieces();
    };
    // A piece is read as the aligned 16-byte chunks it touches, one chunk per lane and load (four neighbours
    // per lane keep the number of load instructions, and of the LDS additions behind them, at a quarter of
    // what one neighbour per lane costs; a compute unit retires such instructions at a fixed pace whatever
    // number of their lanes is active).  The chunks of the batch's pieces are numbered end to end; which
    // piece a chunk belongs to follows from counting piece starts up to it: the starts inside the current
    // span of chunks are bits in LDS, the pieces' records a small table in LDS indexed by their rank among
    // the nonempty ones.  The entries of a piece's first and last chunk that lie outside the piece (the
    // neighbouring windows' or rows') are masked; an aligned 16-byte read that holds at least one entry of
    // the piece stays inside that entry's page.
    struct Span {
        U32x4 v[kAccUnroll];
        uint32_t keep;  // 4 bits per load: which of the 4 entries belong to the piece
        uint32_t chunks;
    };
    Span s0;
    s0.chunks = 0;
    auto more = [&]() { return first < all; };
    auto ask = [&](Span &s) { // the pair's next span, if it has one
        s.keep = s.chunks = 0;
        while (more()) {
            const uint32_t len = bound1 - bound0;
            const int64_t lo_byte = A0 + (row_beg + bound0) * 4, hi_byte = lo_byte + (int64_t)len * 4;
            const int64_t chunk0 = lo_byte & ~(int64_t)15;
            const uint32_t nc = len ? (uint32_t)((hi_byte - 1 - chunk0) >> 4) + 1u : 0u;
            const bool nonempty = nc != 0;
            if (u0 == 0) {
                if (NARROW)
                    have += len;
                const uint32_t inc = wave_inclusive_scan_dpp(nc);
                total = (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
                ustart = inc - nc;
            }
            if (total > u0) {
                s.chunks = min(total - u0, (uint32_t)kAccChunks);
                const uint64_t ne_mask = __ballot(nonempty);
                __builtin_amdgcn_wave_barrier();
                if (nonempty) {
                    AccPiece rec;
                    rec.origin = chunk0 - (int64_t)ustart * 16; // chunk j of the batch starts at origin + 16 j
                    rec.lo = (int32_t)((lo_byte - rec.origin) >> 2);
                    rec.hi = (int32_t)((hi_byte - rec.origin) >> 2);
                    me.piece[bits_below(ne_mask)] = rec;
                }
                if (lane < 2 * kAccUnroll)
                    me.starts[lane] = 0;
                __builtin_amdgcn_wave_barrier();
                const uint32_t rel = ustart - u0; // wraps for pieces that start before the span
                if (nonempty && rel < (uint32_t)kAccChunks)
                    atomicOr(me.starts + (rel >> 5), 1u << (rel & 31u));
                __builtin_amdgcn_wave_barrier();
                int rank = __popcll(__ballot(nonempty && ustart < u0)) - 1; // piece that holds chunk u0 - 1
                uint32_t j0 = (uint32_t)lane;
                asm volatile("" : "+v"(j0)); // (places: computed here, not kept in registers)
#pragma unroll
                for (int u = 0; u < kAccUnroll; ++u) {
                    if ((uint32_t)(u * kWave) >= s.chunks) // (the same for all lanes)
                        break;
                    const uint64_t m = (uint64_t)scalar(reinterpret_cast<const int64_t *>(me.starts)[u]);
                    const int mine = rank + (int)(m & 1u) + (int)bits_below(m >> 1);
                    rank += __popcll(m);
                    if (j0 + u * kWave < s.chunks) {
                        const AccPiece rec = me.piece[mine];
                        const uint32_t x = u0 + j0 + u * kWave; // the lane's chunk, from origin
                        const int from = max(rec.lo - (int)(4 * x), 0), to = min(rec.hi - (int)(4 * x), 4); // its entries in the piece
                        s.v[u] = *reinterpret_cast<const Global<U32x4> *>(rec.origin + (int64_t)x * 16);
                        s.keep |= ((1u << to) - (1u << from)) << (4 * u);
                    }
                }
                __builtin_amdgcn_wave_barrier();
                u0 += kAccChunks;
            }
            if (u0 >= total) { // the next batch's pieces are fetched for the next call
                first += NW * rows;
                fetch_pieces();
            }
            if (s.chunks)
                break;
        }
    };
    // NARROW: all counters of the window in 8 bits (half < 0), or, where that was too little, those of one half of it in 16.
    // (An id's place in the window are its last 16 bits.)
    int half = -1;
    auto add = [&](const Span &s) {
        auto each = [&](auto body) {
#pragma unroll
            for (int u = 0; u < kAccUnroll; ++u) {
                if ((uint32_t)(u * kWave) >= s.chunks)
                    break;
                const U32x4 xs = s.v[u];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if ((s.keep >> (4 * u + e)) & 1u)
                        body(xs[e]);
            }
        };
        if (!NARROW) {
            each([&](uint32_t x) { atomicAdd(&cnt[(x & 0xFFFFu) >> 1], 1u << ((x << 4) & 31u)); });
        } else if (half < 0) {
            each([&](uint32_t x) { atomicAdd(&cnt[(x & 0xFFFFu) >> 2], 1u << ((x << 3) & 31u)); });
        } else {
            each([&](uint32_t x) {
                if ((int)((x >> 15) & 1u) == half)
                    atomicAdd(&cnt[(x & 0x7FFFu) >> 1], 1u << ((x << 4) & 31u));
            });
        }
    };

    uint32_t round = 0, blk = pair_of(0);
    begin_pair(blk);
    ask(s0);
    while (blk < nblk) {
        add(s0);
        while (more()) {
            ask(s0);
            add(s0);
        }
        __syncthreads();
        // A bit per counter in use; lane x of the wave has counters 64 x .. 64 x + 63 of a part, 16 bytes at a time, and
        // begins elsewhere among them than the lanes 2 .. 14 further on: all of LDS's banks have work.
        constexpr int PARTS = NARROW ? 2 : 1; // of the wave; one only of half a window
        const bool bytes = NARROW && half < 0;
        const int parts = bytes ? 2 : 1;
        const uint32_t part0 = bytes ? 2u * (uint32_t)wave : (NARROW && half == 1 ? (uint32_t)NW : 0u) + (uint32_t)wave; // the first, in the window
        uint32_t lane_now = (uint32_t)lane;
        asm volatile("" : "+v"(lane_now)); // (places: computed here, not kept in registers)
        const uint4 *wave4 = reinterpret_cast<const uint4 *>(cnt + wave * kWaveWords);
        uint32_t used[PARTS][2] = {}, w32[PARTS] = {}; // weight: e_v, or e_v^2 of counters of 8 bits
        uint64_t w64 = 0;                              // e_v^2 of counters of 16 bits
        uint32_t shown = 0;                            // e_v
        if (bytes) {
#pragma unroll
            for (int q = 0; q < PARTS; ++q) {
                constexpr int kQuads = kPartIds / 16 / kWave;
                static_assert(kQuads == 4, "64 counters per lane");
#pragma unroll
                for (int it = 0; it < kQuads; ++it) {
                    const uint32_t at = (it + lane_now / 4) & (kQuads - 1);
                    const uint4 v = wave4[q * (kPartIds / 16) + lane_now * kQuads + at];
                    const uint32_t xs[4] = {v.x, v.y, v.z, v.w};
                    uint32_t bits[2] = {0, 0}; // 8 counters each
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const uint32_t nonzero = ((xs[u] & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | xs[u]; // bit 7 of each byte
                        bits[u / 2] = __builtin_amdgcn_udot4((nonzero >> 7) & 0x01010101u, u % 2 ? 0x80402010u : 0x08040201u, bits[u / 2], false);
                        shown = __builtin_amdgcn_sad_u8(xs[u], 0u, shown); // + all four bytes
                        if (SQUARED)
                            w32[q] = __builtin_amdgcn_udot4(xs[u], xs[u], w32[q], false);
                    }
                    const uint32_t both = (bits[0] | bits[1] << 8) << (16 * (at & 1u));
                    used[q][0] |= at < 2 ? both : 0u;
                    used[q][1] |= at < 2 ? 0u : both;
                }
                if (!SQUARED)
                    w32[q] = shown - (q ? w32[0] : 0u);
            }
        } else {
            constexpr int kQuads = kWaveWords / 4 / kWave;
            static_assert(kQuads == 8, "64 counters per lane");
#pragma unroll
            for (int it = 0; it < kQuads; ++it) {
                const uint32_t at = (it + lane_now / 2) & (kQuads - 1);
                const uint4 v = wave4[lane_now * kQuads + at];
                const uint32_t xs[4] = {v.x, v.y, v.z, v.w};
                uint32_t bits = 0; // of the lower counters at 0, 2, 4, 6, of the upper ones at 16, 18, 20, 22
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    bits |= at_most_one(xs[u]) << (2 * u);
                    if (SQUARED) {
                        const uint32_t lo = xs[u] & 0xFFFFu, hi = xs[u] >> 16;
                        w64 += (uint64_t)(lo * lo) + (uint64_t)(hi * hi);
                    } else {
                        w32[0] = __builtin_amdgcn_sad_u16(xs[u], 0u, w32[0]); // + both halves
                    }
                }
                bits = ((bits & 0x55u) | ((bits >> 15) & 0xAAu)) << (8 * (at & 3u));
                used[0][0] |= at < 4 ? bits : 0u;
                used[0][1] |= at < 4 ? 0u : bits;
            }
        }
        uint32_t mine[PARTS], upto[PARTS], part_c[PARTS];
#pragma unroll
        for (int q = 0; q < PARTS; ++q) {
            mine[q] = __popc(used[q][0]) + __popc(used[q][1]);
            upto[q] = wave_inclusive_scan_dpp(mine[q]);
            part_c[q] = (uint32_t)__builtin_amdgcn_readlane((int)upto[q], kWave - 1);
            if (lane == 0 && q < parts)
                sh.cnt[wave * parts + q] = part_c[q];
        }
        if (bytes) {
            const uint32_t missing = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan_dpp(have - shown), kWave - 1);
            if (lane == 0)
                sh.missing[wave] = missing;
        }
        have = 0;
        __syncthreads();
        uint4 *part4 = reinterpret_cast<uint4 *>(cnt + wave * kWaveWords) + lane_now;
        auto clear = [&]() {
#pragma unroll
            for (int it = 0; it < kWaveWords / 4 / kWave; ++it)
                part4[it * kWave] = make_uint4(0, 0, 0, 0);
        };
        // A counter that passed 255 carried into its neighbour or out of its word: that takes 255 or 256 from the sum of all
        // counters, so the sum is that of the neighbours if and only if none did.
        if (bytes && __builtin_amdgcn_readlane((int)wave_inclusive_scan_dpp(lane < NW ? sh.missing[lane] : 0u), NW - 1) != 0) {
            half = 0; // the pair anew, one half after the other
            clear();
            begin_pair(blk);
            ask(s0);
            __syncthreads();
            continue;
        }
        // room for the entries; the parts lie in it one after the other
        const int np = NW * parts;
        const bool as_masks = MASKS && bytes;
        const uint32_t of_part = lane < np ? sh.cnt[lane] : 0u;
        const uint32_t sums = wave_inclusive_scan_dpp(staged_words(of_part, as_masks));
        const uint32_t pair_words = (uint32_t)__builtin_amdgcn_readlane((int)sums, np - 1);
        const uint32_t pair_c = MASKS ? (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan_dpp(of_part), np - 1) : pair_words;
        unsigned long long claim = 0;
        if (tid == 0 && pair_c) {
            unsigned long long *cursor = a.cursor;
            asm volatile("" : "+v"(cursor)); // (an address known to be the same in all lanes has the wave wait for the answer here)
            claim = __hip_atomic_fetch_add((Global<unsigned long long> *)cursor, (unsigned long long)pair_words, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
        }
        const int half_now = half;
        half = half == 0 ? 1 : -1;
        const uint32_t blk_next = half == 1 ? blk : pair_of(++round);
        begin_pair(blk_next);
        // All lanes' counters are listed at once, or, of a part with more in use, those of half of the lanes or of 8 at a time.
        static_assert(8 * 64 <= kAccListed, "8 lanes' counters");
        auto lanes_of = [&](int q) {
            const uint32_t lower = (uint32_t)__builtin_amdgcn_readlane((int)upto[q], kWave / 2 - 1);
            return part_c[q] <= (uint32_t)kAccListed ? kWave : max(lower, part_c[q] - lower) <= (uint32_t)kAccListed ? kWave / 2 : 8;
        };
        auto list_up = [&](int q, int lane0, uint32_t from) { // the lanes' first entry at place 0 of the list: from
            __builtin_amdgcn_wave_barrier();
            if (lane >= lane0 && lane < lane0 + lanes_of(q)) {
                uint16_t *to = me.list + (upto[q] - mine[q] - from);
                for (uint32_t m = used[q][0]; m; m &= m - 1u)
                    *to++ = (uint16_t)(lane * 64 + __ffs((int)m) - 1);
                for (uint32_t m = used[q][1]; m; m &= m - 1u)
                    *to++ = (uint16_t)(lane * 64 + 31 + __ffs((int)m));
            }
            __builtin_amdgcn_wave_barrier();
        };
        list_up(0, 0, 0);
        uint64_t part_w[PARTS], wave_w = 0;
#pragma unroll
        for (int q = 0; q < PARTS; ++q) {
            if (SQUARED && !bytes)
                part_w[q] = q ? 0ull : wave_sum(w64);
            else // (32 bits: 4096 values, below 2^16 or squares of less than 2^8)
                part_w[q] = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan_dpp(w32[q]), kWave - 1);
            wave_w += part_w[q];
        }
        if (tid == 0)
            sh.claimed = claim;
        if (lane == 0)
            atomicAdd(&sh.weight, (unsigned long long)wave_w);
        __syncthreads();
        if (tid == 0) {
            const bool second = NARROW && half_now == 1; // half of the window
            a.win_cnt[blk] = pair_c + (second ? a.win_cnt[blk] : 0u);
            a.win_wt[blk] = sh.weight + (second ? a.win_wt[blk] : 0ull);
            sh.weight = 0; // (two barriers before the next pair's)
        }
        const int64_t claimed = scalar((int64_t)sh.claimed);
#pragma unroll
        for (int q = 0; q < PARTS; ++q) {
            if (q >= parts)
                continue;
            const bool masks = as_masks && part_c[q] >= kMaskFrom;
            const int64_t base = claimed + (uint32_t)__builtin_amdgcn_readlane((int)sums, wave * parts + q) - staged_words(part_c[q], as_masks);
            if (lane == 0) {
                const int64_t part = (int64_t)blk * kWinParts + part0 + q;
                a.part_base[part] = 2 * base + (masks ? 1 : 0);
                a.part_cnt[part] = part_c[q];
                a.part_wt[part] = part_w[q];
            }
            if (part_c[q] == 0)
                continue;
            uint32_t *__restrict__ out = a.tmp_ent + base;
            const uint16_t *cnt16 = reinterpret_cast<const uint16_t *>(wave4);
            const uint8_t *cnt8 = reinterpret_cast<const uint8_t *>(wave4 + q * (kPartIds / 16));
            const uint32_t part_id = (part0 + q) * kPartIds;
            const int lanes = lanes_of(q);
            if (masks) {
                U32x2_a4 bits;
                bits.x = used[q][0];
                bits.y = used[q][1];
                reinterpret_cast<U32x2_a4 *>(out)[lane] = bits;
                uint32_t *__restrict__ bytes_out = out + kMaskWords;
                uint32_t left = 0; // a place of those listed before that do not fill a word, by lane
                for (int lane0 = 0; lane0 < kWave; lane0 += lanes) {
                    const uint32_t listed = lane0 ? (uint32_t)__builtin_amdgcn_readlane((int)upto[q], lane0 - 1) : 0u;
                    const uint32_t upto_here = (uint32_t)__builtin_amdgcn_readlane((int)upto[q], lane0 + lanes - 1);
                    const uint32_t from = listed & ~3u, n = upto_here - from; // places in the list
                    if (lane0 || q)
                        list_up(q, lane0, from);
                    if ((uint32_t)lane < (listed & 3u))
                        me.list[lane] = (uint16_t)left;
                    __builtin_amdgcn_wave_barrier();
                    const bool end = lane0 + lanes == kWave;
                    const uint32_t words = end ? (n + 3u) / 4u : n / 4u;
                    for (uint32_t x = lane; x < words; x += kWave) {
                        // (behind the last entry there is anything in the list)
                        const uint64_t ids = reinterpret_cast<const FourPlaces *>(me.list)[x];
                        uint32_t word = 0;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            word |= (uint32_t)cnt8[(uint32_t)(ids >> (16 * e)) & (kPartIds - 1u)] << (8 * e);
                        bytes_out[from / 4u + x] = word;
                    }
                    if (!end)
                        left = me.list[(n & ~3u) + (lane & 3u)]; // (three places behind the list's end at most: it has them)
                }
                continue;
            }
            for (int lane0 = 0; lane0 < kWave; lane0 += lanes) {
                const uint32_t listed = lane0 ? (uint32_t)__builtin_amdgcn_readlane((int)upto[q], lane0 - 1) : 0u;
                const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)upto[q], lane0 + lanes - 1) - listed;
                if (lane0 || q)
                    list_up(q, lane0, listed);
                auto leave = [&](auto *counters) {
                    for (uint32_t x0 = lane; x0 < n; x0 += kAccFlush * kWave) {
                        uint32_t id[kAccFlush], c[kAccFlush];
#pragma unroll
                        for (int u = 0; u < kAccFlush; ++u)
                            id[u] = me.list[min(x0 + u * kWave, n - 1u)];
#pragma unroll
                        for (int u = 0; u < kAccFlush; ++u)
                            c[u] = counters[id[u]];
#pragma unroll
                        for (int u = 0; u < kAccFlush; ++u)
                            if (x0 + u * kWave < n)
                                out[listed + x0 + u * kWave] = (part_id + id[u]) << 16 | c[u];
                    }
                };
                if (bytes)
                    leave(cnt8);
                else
                    leave(cnt16);
            }
        }
        __builtin_amdgcn_wave_barrier();
        clear(); // the next pair begins at zero
        ask(s0); // of the next pair
        __syncthreads();
        blk = blk_next;
    }
}

// A hop whose parts may be masks: kernels of their own, whose longer code the others need not run through
struct LwMasks {
    LwHop hop;
};
template <bool SQUARED, bool NARROW>
__global__ __launch_bounds__(kAccThreads<NARROW>, 4) void ldw_accumulate_kernel(LwHop a) { accumulate<SQUARED, NARROW, false>(a); }
template <bool SQUARED, bool NARROW>
__global__ __launch_bounds__(kAccThreads<NARROW>, 4) void ldw_accumulate_kernel(LwMasks a) { accumulate<SQUARED, NARROW, true>(a.hop); }

// Workgroups 0 .. k - 1, one per minibatch: columns and weight before each part of every window, and before each window; columns
// and weight of the minibatch.  A part per thread, so 16 lanes per window.  The others plan (plan_tiles).
// Three layers of 32 x 512 seeds, 37 windows: 26 us with a window per thread, which read its 16 parts one after the other, 20 so.
constexpr int kScanThreads = 1024;
__global__ __launch_bounds__(kScanThreads) void ldw_win_scan_kernel(LwHop a, int64_t *pnnz_out)
{
    static_assert(kWinParts == 16, "a window's parts are 16 lanes");
    __shared__ uint64_t smem[kScanThreads / kWave];
    __shared__ uint32_t smem_c[kScanThreads / kWave];
    __shared__ uint32_t last_s;
    __shared__ PlanShared plan;
    if ((int)blockIdx.x >= a.k) {
        if (!(a.giveup && *a.giveup)) // (it went up before this launch or not at all)
            plan_tiles<kScanThreads>(a, plan, reinterpret_cast<int64_t *>(smem), (int)blockIdx.x - a.k, (int)gridDim.x - a.k);
        return;
    }
    const int i = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    // the workgroup that comes here last turns the minibatches' counts into p_off
    auto finish = [&](int64_t count) {
        if (tid == 0) {
            __hip_atomic_store(a.mb_count + i, count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            last_s = arrive_last(a.done, (uint32_t)a.k) ? 1u : 0u;
        }
        __syncthreads();
        if (!last_s)
            return;
        uint64_t carry = 0;
        for (int32_t base = 0; base < a.k; base += kScanThreads) {
            const int32_t j = base + tid;
            const uint64_t v = j < a.k ? (uint64_t)__hip_atomic_load(a.mb_count + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
            uint64_t total;
            const uint64_t ex = carry + block_exclusive_scan<uint64_t, kScanThreads>(v, smem, total);
            if (j < a.k)
                a.p_off[j] = (int64_t)ex;
            carry += total;
        }
        if (tid == 0) {
            a.p_off[a.k] = (int64_t)carry;
            *pnnz_out = (int64_t)carry;
        }
    };
    if (a.giveup && *a.giveup) {
        finish(0);
        return;
    }
    uint64_t carry_c = 0, carry_w = 0;
    const int32_t parts = a.nwin * kWinParts;
    const int64_t first = (int64_t)i * parts;
    for (int32_t base = 0; base < parts; base += kScanThreads) {
        const int32_t q = base + tid;
        const uint32_t c = q < parts ? a.part_cnt[first + q] : 0u; // of one minibatch, so all of them are no more than n
        const uint64_t wt = q < parts ? a.part_wt[first + q] : 0ull;
        const uint32_t upto_c = wave_inclusive_scan_dpp(c);
        const uint64_t upto_w = wave_inclusive_scan(wt);
        __syncthreads(); // the sums of the steps before have been read
        if (lane == kWave - 1) {
            smem_c[wave] = upto_c;
            smem[wave] = upto_w;
        }
        __syncthreads();
        uint64_t before_c = carry_c, before_w = carry_w;
#pragma unroll
        for (int x = 0; x < kScanThreads / kWave; ++x) {
            before_c += x < wave ? smem_c[x] : 0u;
            before_w += x < wave ? smem[x] : 0ull;
            carry_c += smem_c[x];
            carry_w += smem[x];
        }
        const int head = lane & ~(kWinParts - 1);
        const uint32_t head_c = (uint32_t)__shfl((int)(upto_c - c), head, kWave);
        const uint64_t head_w = __shfl(upto_w - wt, head, kWave);
        if (q < parts) {
            a.part_off[first + q] = upto_c - c - head_c;
            a.part_woff[first + q] = upto_w - wt - head_w;
            const int64_t x = (first + q) / kWinParts;
            if (lane == head) {
                a.win_poff[x] = (int64_t)(before_c + head_c);
                a.win_woff[x] = before_w + head_w;
            }
        }
    }
    if (tid == 0)
        a.mb_wt[i] = carry_w;
    finish((int64_t)carry_c);
}

// A part to its place in P with the inclusive prefix sums of the weights, by one wave: `cw` entries at src, 64 at a time, with lane
// scans for the sums and no workgroup barrier.  carry: weight of the minibatch before the part.
constexpr int kCopyUnroll = 4;
__device__ inline void fetch_entries(const uint32_t *__restrict__ src, uint32_t x0, uint32_t cw, uint32_t (&ent)[kCopyUnroll])
{
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) {
        const uint32_t x = x0 + u * kWave + (threadIdx.x & (kWave - 1));
        ent[u] = x < cw ? src[x] : 0u;
    }
}
template <bool SQUARED, bool PAST>
__device__ inline void place_entries(const LwHop &a, const uint32_t (&ent)[kCopyUnroll], uint32_t x0, uint32_t cw, int64_t dst, int32_t id0,
                                     uint64_t &carry)
{
    const int64_t first = scalar(dst + (int32_t)x0); // (places in scalar registers and offsets that are constants)
    int32_t *col = a.p_col + first;
    uint32_t *cnt = a.p_cnt + first;
    const uint32_t lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) {
        const uint32_t c = ent[u] & 0xFFFFu;
        // e_v < 2^16: sums of 64 weights e_v fit 32 bits; e_v^2 is summed as two 16-bit halves
        uint64_t inc;
        if (SQUARED) {
            const uint32_t wq = c * c;
            inc = ((uint64_t)wave_inclusive_scan_dpp(wq >> 16) << 16) + wave_inclusive_scan_dpp(wq & 0xFFFFu);
        } else {
            inc = wave_inclusive_scan_dpp(c);
        }
        if (x0 + u * kWave + lane < cw) {
            if (PAST) { // the caches (LwHop::p_past)
                __builtin_nontemporal_store(id0 + (int32_t)(ent[u] >> 16), col + u * kWave + lane);
                __builtin_nontemporal_store(c, cnt + u * kWave + lane);
            } else {
                col[u * kWave + lane] = id0 + (int32_t)(ent[u] >> 16);
                cnt[u * kWave + lane] = c;
            }
            // the draws find their block of kPrefixBlock entries of P by these sums and walk the weights
            // inside it: only the sum at the last entry of every such block (absolute index in P) is kept
            const int64_t at = first + u * kWave + lane;
            if ((at & (kPrefixBlock - 1)) == kPrefixBlock - 1)
                a.prefix[at / kPrefixBlock] = carry + inc;
        }
        carry += (uint64_t)lane_value((int64_t)inc, kWave - 1);
    }
}

// A wave's view of a part in masks, up to kCopyListed entries at a time: the columns and e_v of those at places 32 w .. of P, where the first
// of them lies in the 32 places (a memory line) from place 0 on
constexpr uint32_t kCopyListed = 992;
struct CopyWave {
    alignas(16) uint8_t cnt[kCopyListed + 32];
    uint16_t list[kCopyListed + 32];
};
using U16_any = uint16_t __attribute__((may_alias));
using U32_any = uint32_t __attribute__((may_alias));
using U32x4_any = uint32_t __attribute__((ext_vector_type(4), may_alias));
using U32x4_a1 = uint32_t __attribute__((ext_vector_type(4), aligned(1)));
constexpr int64_t kMostCopying = 1 << 18; // workgroups (a launch has fewer than 2^32 threads)
template <bool PAST, class T>
__device__ inline void store_p(T x, T *to) // PAST: past the caches (LwHop::p_past)
{
    if (PAST)
        __builtin_nontemporal_store(x, to);
    else
        *to = x;
}

// Many pairs: a window left the accumulation in kWinParts parts whose places are on record (ldw_win_scan).  Whole lines of P
// to a store: a wave's first 32 places are those of the line that the part begins in.
//   MASKS  (LwHop::p_masks: parts hold many entries, most of them in masks) a part per wave (above 65536 pairs several), started in the
//          order of P: what the chip writes at a time then lies close together, and the next workgroups fill the waits.  All e_v of a part (of up to
//          kCopyListed entries) are read before the first store (a load that is asked for behind stores is only there when they are done),
//          and a lane has two entries: half the stores and lane scans.  115 M entries, 8.7 M vertices, all of the call's hops (3 GB with
//          parts as entries, 2.6 with masks): 688 us with 17 parts a wave, one after the other and 64 entries to a store; 620 from masks, 587 by
//          two entries a lane and reads ahead of stores, 531 with 2 parts a wave, 509 with one (5.1 TB/s).
//   else   eight workgroups per compute unit that go from part to part: of parts of a few entries a launch of a wave each costs more than the
//          waits, and their records are read by the vector unit, which has more reads on their way than the scalar one.  64 x 64 seeds, two
//          hops, 4 and 50 entries a part: 94 us by the kernel for masks, 80 so; 200 x 256 on 2.4 M vertices, 21 entries: 42 and 36; ids by descending
//          degree, 64 x 256, 3 and 39 entries: 107 and 72.  The records by the vector unit with masks: 437 -> 457 us of three layers of 64 x 1024.
template <bool MASKS, class T>
__device__ inline T part_record(const T *p)
{
    if constexpr (MASKS)
        return uniform_load(p);
    else if constexpr (sizeof(T) == 4)
        return (T)scalar((uint32_t)*p);
    else
        return (T)scalar((int64_t)*p);
}
template <bool SQUARED, bool PAST, bool MASKS>
__device__ __forceinline__ void copy_parts(const LwHop &a)
{
    __shared__ CopyWave waves[MASKS ? 256 / kWave : 1];
    if (a.giveup) {
        if (*a.giveup)
            return;
        if (a.p_off[a.k] > a.p_cap) { // P does not fit what was provided (the same in every workgroup)
            if (blockIdx.x == 0 && threadIdx.x == 0)
                *a.giveup = 1;
            return;
        }
    }
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = scalar(threadIdx.x / kWave);
    CopyWave &me = waves[MASKS ? wave : 0];
    const int64_t nparts = (int64_t)a.k * a.nwin * kWinParts;
    for (int64_t part = (int64_t)blockIdx.x * (256 / kWave) + wave; part < nparts; part += (int64_t)gridDim.x * (256 / kWave)) {
        const uint32_t cw = part_record<MASKS>(a.part_cnt + part);
        if (cw == 0)
            continue;
        const int64_t blk = part / kWinParts;
        const int32_t i = (int32_t)((uint32_t)blk / (uint32_t)a.nwin); // (at most 2^16 minibatches and 2^15 windows)
        const int32_t window = (int32_t)blk - i * a.nwin;
        const int64_t base = part_record<MASKS>(a.part_base + part);
        const int64_t dst = part_record<MASKS>(a.p_off + i) + part_record<MASKS>(a.win_poff + blk) + part_record<MASKS>(a.part_off + part);
        uint64_t carry = part_record<MASKS>(a.win_woff + blk) + part_record<MASKS>(a.part_woff + part);
        const uint32_t *__restrict__ src = a.tmp_ent + (base >> 1);
        if (!MASKS || !(base & 1)) {
            for (int32_t x0 = -(int32_t)(dst & 31); x0 < (int32_t)cw; x0 += kCopyUnroll * kWave) {
                uint32_t ent[kCopyUnroll];
                fetch_entries(src, (uint32_t)x0, cw, ent);
                place_entries<SQUARED, PAST>(a, ent, (uint32_t)x0, cw, dst, window << kWinShift, carry);
            }
            continue;
        }
        const uint32_t id0 = (uint32_t)window << kWinShift | (uint32_t)(part % kWinParts) * kPartIds;
        // e_v of the entries from `from` on, and of the places before them in their line of P
        auto fetch_counts = [&](uint32_t from) {
            const uint32_t head = (uint32_t)(dst + from) & 31u;
            const uint8_t *counts = reinterpret_cast<const uint8_t *>(src + kMaskWords) + from;
            U32x4_a1 x = {0, 0, 0, 0};
            if (16 * lane < cw - from + head) // (up to 15 bytes behind the part, which is 64 words shorter than the room there is for it)
                x = *reinterpret_cast<const U32x4_a1 *>(counts + ((int32_t)(16 * lane) - (int32_t)head));
            return x;
        };
        const U32x2_a4 bits = reinterpret_cast<const U32x2_a4 *>(src)[lane]; // 64 columns a lane
        U32x4_a1 counts = fetch_counts(0);
        const uint32_t used = __popc(bits.x) + __popc(bits.y), upto = wave_inclusive_scan_dpp(used);
        const uint32_t lower = (uint32_t)__builtin_amdgcn_readlane((int)upto, kWave / 2 - 1);
        static_assert(8 * 64 <= kCopyListed, "8 lanes' columns");
        const uint32_t lanes = cw <= kCopyListed ? kWave : max(lower, cw - lower) <= kCopyListed ? kWave / 2 : 8;
        for (uint32_t lane0 = 0; lane0 < kWave; lane0 += lanes) {
            const uint32_t from = lane0 ? (uint32_t)__builtin_amdgcn_readlane((int)upto, (int)lane0 - 1) : 0u;
            const uint32_t to = (uint32_t)__builtin_amdgcn_readlane((int)upto, (int)(lane0 + lanes) - 1), n = to - from;
            const uint32_t head = (uint32_t)(dst + from) & 31u;
            __builtin_amdgcn_wave_barrier();
            reinterpret_cast<U32x4_any *>(me.cnt)[lane] = counts;
            if (lane - lane0 < lanes) {
                uint16_t *to_lo = me.list + head + (upto - used - from), *to_hi = to_lo + __popc(bits.x);
                const uint32_t id = lane * 64u;
                for (uint32_t lo = bits.x, hi = bits.y; lo | hi;) {
                    if (lo) {
                        *to_lo++ = (uint16_t)(id + (uint32_t)__ffs((int)lo) - 1u);
                        lo &= lo - 1u;
                    }
                    if (hi) {
                        *to_hi++ = (uint16_t)(id + (uint32_t)__ffs((int)hi) + 31u);
                        hi &= hi - 1u;
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
            if (lane0 + lanes < kWave)
                counts = fetch_counts(to);
            const int64_t line = scalar(dst + from - head); // a multiple of 32
            for (uint32_t x = 0; x < head + n; x += 2 * kWave) {
                const uint32_t y = x + 2 * lane;
                const uint32_t ids = *reinterpret_cast<const U32_any *>(me.list + y);
                const uint32_t both = *reinterpret_cast<const U16_any *>(me.cnt + y);
                const bool in0 = y - head < n, in1 = y + 1u - head < n;
                const uint32_t c0 = in0 ? both & 0xFFu : 0u, c1 = in1 ? both >> 8 : 0u;
                const uint32_t inc = wave_inclusive_scan_dpp(SQUARED ? c0 * c0 + c1 * c1 : c0 + c1); // (128 weights of less than 2^16)
                int32_t *col = a.p_col + line + x;
                uint32_t *cnt = a.p_cnt + line + x;
                const int32_t v0 = (int32_t)(id0 + (ids & 0xFFFFu)), v1 = (int32_t)(id0 + (ids >> 16));
                if (in0 && in1) {
                    const I32x2_a4 v = {v0, v1};
                    const U32x2_a4 c = {c0, c1};
                    store_p<PAST>(v, reinterpret_cast<I32x2_a4 *>(col) + lane);
                    store_p<PAST>(c, reinterpret_cast<U32x2_a4 *>(cnt) + lane);
                } else if (in0 || in1) {
                    const uint32_t at = 2 * lane + (in0 ? 0u : 1u);
                    store_p<PAST>(in0 ? v0 : v1, col + at);
                    store_p<PAST>(in0 ? c0 : c1, cnt + at);
                }
                if (in1 && (lane & 7u) == 7u) // the last of kPrefixBlock entries
                    a.prefix[(line + x + 2 * lane) / kPrefixBlock] = carry + inc;
                carry += (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
            }
        }
    }
}
template <bool SQUARED, bool PAST>
__global__ __launch_bounds__(256) void ldw_p_copy_kernel(LwHop a) { copy_parts<SQUARED, PAST, false>(a); }
template <bool SQUARED, bool PAST>
__global__ __launch_bounds__(256) void ldw_p_copy_kernel(LwMasks a) { copy_parts<SQUARED, PAST, true>(a.hop); }

// Up to kMostPlacedPairs pairs: scan, copy and plan in one launch.  The first `planners` workgroups plan, each of the others takes a
// pair and adds up the sizes of those before it (P is stacked like the pairs) while the entries are on their way.
constexpr int kMostPlacedPairs = 2048;
template <bool SQUARED, int NT>
__global__ __launch_bounds__(NT) void ldw_p_place_kernel(LwHop a, int planners, int64_t *pnnz_out)
{
    constexpr int NW = NT / kWave, EACH = kWinParts / NW; // parts per wave
    __shared__ PlanShared plan;
    __shared__ int64_t smem[NW];
    __shared__ uint64_t smem_w[NW];
    __shared__ int32_t up_s; // the flag as this workgroup sees it: it may go up meanwhile
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = (int)scalar((uint32_t)tid / kWave);
    if (tid == 0)
        up_s = a.giveup ? *a.giveup : 0;
    __syncthreads();
    if (up_s)
        return;
    if ((int)blockIdx.x < planners) {
        plan_tiles<NT>(a, plan, smem, (int)blockIdx.x, planners);
        return;
    }
    const uint32_t pair = blockIdx.x - (uint32_t)planners, i = pair / (uint32_t)a.nwin, head = i * (uint32_t)a.nwin;
    const int64_t part0 = (int64_t)pair * kWinParts;
    const uint32_t cnt = lane < kWinParts ? a.part_cnt[part0 + lane] : 0u;
    const uint64_t wt = lane < kWinParts ? a.part_wt[part0 + lane] : 0ull;
    const int64_t base = lane < kWinParts ? a.part_base[part0 + lane] : 0;
    uint32_t c = 0; // of all pairs: fewer than 2^32
    uint64_t w = 0;
#pragma unroll
    for (uint32_t q = tid; q < (uint32_t)kMostPlacedPairs; q += NT)
        if (q < pair) {
            c += a.win_cnt[q];
            w += q >= head ? a.win_wt[q] : 0ull;
        }
    uint32_t ent[EACH][kCopyUnroll];
#pragma unroll
    for (int e = 0; e < EACH; ++e) {
        const int q = wave * EACH + e;
        fetch_entries(a.tmp_ent + (lane_value(base, q) >> 1), 0, (uint32_t)__builtin_amdgcn_readlane((int)cnt, q), ent[e]);
    }
    const uint32_t upto_c = wave_inclusive_scan_dpp(cnt);
    const uint64_t upto_w = wave_inclusive_scan(wt);
    const uint32_t pair_c = (uint32_t)__builtin_amdgcn_readlane((int)upto_c, kWinParts - 1);
    const uint64_t pair_w = (uint64_t)lane_value((int64_t)upto_w, kWinParts - 1);
    const uint32_t wave_c = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan_dpp(c), kWave - 1);
    const uint64_t wave_w = wave_sum(w);
    if (lane == 0) {
        smem[wave] = wave_c;
        smem_w[wave] = wave_w;
    }
    __syncthreads();
    int64_t before = 0;
    uint64_t before_w = 0;
#pragma unroll
    for (int x = 0; x < NW; ++x) {
        before += smem[x];
        before_w += smem_w[x];
    }
    if (tid == 0) {
        if (pair == head)
            a.p_off[i] = before;
        if (pair == head + (uint32_t)a.nwin - 1u)
            a.mb_wt[i] = before_w + pair_w;
        if (pair == (uint32_t)a.k * (uint32_t)a.nwin - 1u) {
            a.p_off[a.k] = before + pair_c;
            *pnnz_out = before + pair_c;
        }
    }
    if (a.giveup && before + pair_c > a.p_cap) { // P does not fit what was provided
        if (tid == 0)
            *a.giveup = 1;
        return;
    }
    const int32_t id0 = (int32_t)(pair - head) << kWinShift;
#pragma unroll
    for (int e = 0; e < EACH; ++e) {
        const int q = wave * EACH + e;
        const uint32_t cw = (uint32_t)__builtin_amdgcn_readlane((int)cnt, q);
        if (cw == 0)
            continue;
        const uint32_t *__restrict__ src = a.tmp_ent + (lane_value(base, q) >> 1);
        const int64_t dst = before + (uint32_t)__builtin_amdgcn_readlane((int)(upto_c - cnt), q);
        uint64_t carry = before_w + (uint64_t)lane_value((int64_t)(upto_w - wt), q);
        place_entries<SQUARED, false>(a, ent[e], 0, cw, dst, id0, carry);
        for (uint32_t x0 = kCopyUnroll * kWave; x0 < cw; x0 += kCopyUnroll * kWave) {
            uint32_t more[kCopyUnroll];
            fetch_entries(src, x0, cw, more);
            place_entries<SQUARED, false>(a, more, x0, cw, dst, id0, carry);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// SAMPLE: one workgroup per minibatch, or several
// ---------------------------------------------------------------------------------------------
constexpr int kDrawThreads = 1024;
// The value of lane ^ X: by the vector unit where it can, else through LDS's crossbar
template <int X>
__device__ inline uint32_t lane_xor(uint32_t v)
{
    if (X == 1)
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1 /* quad_perm:[1,0,3,2] */, 0xF, 0xF, true);
    if (X == 2)
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E /* quad_perm:[2,3,0,1] */, 0xF, 0xF, true);
    if (X == 8)
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128 /* row_ror:8 */, 0xF, 0xF, true);
    return __shfl_xor(v, X, kWave);
}

// Bitonic sort, ascending, of the first n of PER x 1024 places (the rest hold kEmptySlot): thread t holds places t, t + 1024, ...
// Partners in the thread itself and in its wave need no barrier; of the 55 steps for 1024 keys 10 go through LDS (ex: two buffers
// in turn, PER x 1024 words each).
template <int PER, int SIZE, int STRIDE>
__device__ inline void sort_step(uint32_t (&key)[PER], int n, uint32_t *ex, int &turn)
{
    const uint32_t tid = threadIdx.x;
    uint32_t other[PER];
    if (STRIDE >= kDrawThreads) {
#pragma unroll
        for (int q = 0; q < PER; ++q)
            other[q] = key[(q ^ (STRIDE / kDrawThreads)) % PER];
    } else if (STRIDE >= kWave) {
        uint32_t *to = ex + turn * PER * kDrawThreads;
#pragma unroll
        for (int q = 0; q < PER; ++q)
            to[q * kDrawThreads + tid] = key[q];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; ++q)
            other[q] = to[q * kDrawThreads + (tid ^ (uint32_t)STRIDE)];
        turn ^= 1;
    } else {
#pragma unroll
        for (int q = 0; q < PER; ++q)
            other[q] = lane_xor<STRIDE < kWave ? STRIDE : 1>(key[q]);
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const uint32_t at = (uint32_t)(q * kDrawThreads) + tid;
        const bool low = ((at & (uint32_t)STRIDE) == 0) == ((at & (uint32_t)SIZE) == 0);
        key[q] = low ? min(key[q], other[q]) : max(key[q], other[q]);
    }
    if constexpr (STRIDE > 1)
        sort_step<PER, SIZE, STRIDE / 2>(key, n, ex, turn);
    else if constexpr (SIZE < PER * kDrawThreads)
        if (SIZE < n)
            sort_step<PER, SIZE * 2, SIZE>(key, n, ex, turn);
}

// N draws of a thread: the smallest entries of P (absolute index) whose sums in the minibatch exceed r[]; side by side, as each is
// a chain of trips to memory.  pre: recorded sums of the nb blocks that end in the minibatch's row [p0, p0 + C); top: the sums at
// the ends of the ntop groups of 2^st blocks; pnnz >= 16.
struct DrawRow {
    int64_t p0, C, B0, nb, ntop, pnnz;
    const uint64_t *pre;
    int st, squared;
};
template <int N>
__device__ inline void find_entries(const LwHop &a, const DrawRow &d, const uint64_t *top, const uint64_t (&r)[N], int64_t (&e)[N])
{
    int64_t pos[N]; // groups, then blocks, whose sums do not exceed r
#pragma unroll
    for (int x = 0; x < N; ++x)
        pos[x] = 0;
#pragma unroll
    for (int step = kDrawTop; step > 0; step >>= 1)
#pragma unroll
        for (int x = 0; x < N; ++x) {
            const int64_t at = pos[x] + step;
            if (at <= d.ntop && top[at <= d.ntop ? at - 1 : 0] <= r[x])
                pos[x] = at;
        }
#pragma unroll
    for (int x = 0; x < N; ++x)
        pos[x] <<= d.st;
    for (int w = d.st; w > 0;) { // three bits of the place in the group at a time: 7 sums in flight
        const int bits = min(w, 3);
        w -= bits;
        uint64_t sum[N][7];
#pragma unroll
        for (int x = 0; x < N; ++x)
#pragma unroll
            for (int i = 0; i < 7; ++i) {
                const int64_t at = pos[x] + ((int64_t)(i + 1) << w) - 1;
                sum[x][i] = i + 1 < 1 << bits && at < d.nb ? d.pre[at] : ~0ull;
            }
#pragma unroll
        for (int x = 0; x < N; ++x) {
            int n = 0;
#pragma unroll
            for (int i = 0; i < 7; ++i)
                n += sum[x][i] <= r[x] ? 1 : 0;
            pos[x] += (int64_t)n << w;
        }
    }
    // the 16 entries of the block (the minibatch's ones among them): the last block of all is read from 16 entries before its end
    using Four = uint32_t __attribute__((ext_vector_type(4), aligned(4)));
    uint64_t acc[N];
    Four v[N][kPrefixBlock / 4];
    int64_t from[N];
#pragma unroll
    for (int x = 0; x < N; ++x) {
        acc[x] = pos[x] > 0 ? d.pre[pos[x] - 1] : 0ull;
        e[x] = (d.B0 + pos[x]) * kPrefixBlock;
        from[x] = min<int64_t>(e[x], d.pnnz - kPrefixBlock);
#pragma unroll
        for (int i = 0; i < kPrefixBlock / 4; ++i)
            v[x][i] = *reinterpret_cast<const Four *>(a.p_cnt + from[x] + 4 * i);
    }
    const int64_t end = d.p0 + d.C - 1; // the smallest t with prefix[t] > r exists below the row's end: W > r
#pragma unroll
    for (int x = 0; x < N; ++x) {
        const int32_t first = (int32_t)(max(e[x], d.p0) - from[x]), last = (int32_t)min<int64_t>(end - from[x], kPrefixBlock);
        int32_t n = 0; // of the entries first .. last - 1 those whose sums do not exceed r
#pragma unroll
        for (int i = 0; i < kPrefixBlock; ++i) {
            const uint32_t c = i >= first ? v[x][i / 4][i % 4] : 0u;
            acc[x] += d.squared ? (uint64_t)c * c : (uint64_t)c;
            n += i >= first && i < last && acc[x] <= r[x] ? 1 : 0;
        }
        e[x] = from[x] + first + n;
    }
}

// The entry of one draw, where P has fewer than 16
__device__ inline int64_t walk_entries(const LwHop &a, const DrawRow &d, uint64_t r)
{
    int64_t e = d.p0;
    for (uint64_t acc = ldw_weight(a.p_cnt[e], a.squared); acc <= r; acc += ldw_weight(a.p_cnt[e], a.squared))
        ++e;
    return e;
}

// PLACE: the sampled columns go to their place in the stack at once, behind those of the minibatches before (sum_before).
// PER: places of the sort per thread, 1024 PER >= s.  A chain of trips to memory and barriers on one compute unit: the
// draws of a thread search side by side, the 16 entries of a block arrive together, and most steps of the sort need no barrier.
// 3 minibatches, 512 draws: 21 -> 9 us (sort 11 -> 2.5, entries of a block one by one 3 -> 1).  64 minibatches, 2048 draws from
// 115 thousand blocks: 75 -> 71 us; there the sums and entries looked up, some 14 thousand lines per compute unit, are the bound
// (50 us of it, whatever their order), and the sort went from 16 to 5 us.
// SHARED (with PLACE): `parts` workgroups of a minibatch find a share of its draws each, and the one that is done last sorts and places
// them all (launch_ldw_draw): 71 -> 42 us, four of them.
template <bool PLACE, int PER, bool SHARED>
__global__ __launch_bounds__(kDrawThreads) void ldw_draw_kernel(LwHop a, Lookback lb, int64_t *ncols_out, int parts)
{
    __shared__ uint32_t ex[2 * PER * kDrawThreads];
    __shared__ uint64_t top[kDrawTop];
    __shared__ int64_t smem64[kDrawThreads / kWave];
    __shared__ uint32_t heads_of[PER * kDrawThreads / kWave];
    __shared__ uint32_t number_s;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int number = PLACE ? (int)scalar(take_number(lb, &number_s)) : (int)blockIdx.x;
    // (in the order of starting: who places waits only for minibatches all of whose workgroups have started)
    const int i = SHARED ? number / parts : number, part = SHARED ? number - i * parts : 0;
    // where the minibatch's `count` columns begin
    auto place = [&](uint32_t count) {
        const int64_t before = sum_before<kDrawThreads>(lb, (uint32_t)i, count, smem64);
        if (tid == 0) {
            a.mb_coloff[i] = before;
            if (i == a.k - 1) {
                a.mb_coloff[a.k] = before + count;
                *ncols_out = before + count;
            }
        }
        return before;
    };
    DrawRow d;
    d.pnnz = uniform_load(a.p_off + a.k);
    if (a.giveup && (uniform_load(a.giveup) || d.pnnz > a.p_cap)) { // no P: the minibatch gets no columns
        if (PLACE) {
            if (part == 0)
                place(0);
        } else if (tid == 0)
            a.mb_count[i] = 0;
        return;
    }
    d.p0 = uniform_load(a.p_off + i);
    d.C = uniform_load(a.p_off + i + 1) - d.p0;
    // inclusive weight sums are on record at the last entry of every block of kPrefixBlock entries (absolute
    // index in P): blocks B0 .. B0 + nb - 1 end inside this minibatch's row; W = the row sum
    d.B0 = d.p0 / kPrefixBlock;
    d.nb = (d.p0 + d.C) / kPrefixBlock - d.B0;
    d.pre = a.prefix + d.B0;
    d.squared = a.squared;
    const uint64_t W = uniform_load(a.mb_wt + i);
    const uint64_t rk = row_key(a.hopkey, a.mb_base + (uint32_t)i, kNoVertex);
    // Every draw searches the recorded sums.  Those at the end of every group of 2^st blocks (at most kDrawTop groups) are copied
    // to LDS first: a draw finds its group there and only the last st bits are looked for in memory.
    d.st = 0;
    while ((d.nb >> d.st) > kDrawTop)
        ++d.st;
    d.ntop = d.nb >> d.st;
    uint64_t sums[kDrawTop / kDrawThreads];
#pragma unroll
    for (int q = 0; q < kDrawTop / kDrawThreads; ++q) {
        const int64_t t = q * kDrawThreads + tid;
        sums[q] = t < d.ntop ? d.pre[((t + 1) << d.st) - 1] : 0ull;
    }
#pragma unroll
    for (int q = 0; q < kDrawTop / kDrawThreads; ++q)
        top[q * kDrawThreads + tid] = sums[q];
    __syncthreads();
    uint32_t key[PER];
    if (SHARED) {
        int32_t *__restrict__ found = a.sel_tmp + (int64_t)i * a.s;
        const int each = (a.s + parts - 1) / parts, end = min((part + 1) * each, a.s);
        for (int j = part * each + tid; j < end; j += kDrawThreads) {
            const uint64_t r[1] = {bounded64(draw64(rk, (uint32_t)j), W)};
            uint32_t column = kEmptySlot;
            if (d.C > 0) {
                int64_t e[1];
                if (d.pnnz >= kPrefixBlock)
                    find_entries<1>(a, d, top, r, e);
                else
                    e[0] = walk_entries(a, d, r[0]);
                column = (uint32_t)a.p_col[e[0]];
            }
            __hip_atomic_store(found + j, (int32_t)column, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // what each wave found is where other dies see it
        __syncthreads();
        if (tid == 0)
            number_s = arrive_last(a.draw_done + i, (uint32_t)parts) ? 1u : 0u;
        __syncthreads();
        if (!number_s)
            return;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int j = q * kDrawThreads + tid;
            key[q] = j < a.s ? (uint32_t)__hip_atomic_load(found + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : kEmptySlot;
        }
    } else if (d.C > 0 && d.pnnz >= kPrefixBlock) {
        constexpr int N = PER < 2 ? PER : 2; // draws side by side
#pragma unroll
        for (int q = 0; q < PER; q += N) {
#pragma unroll
            for (int x = 0; x < N; ++x)
                key[q + x] = kEmptySlot;
            if (q * kDrawThreads + (int)scalar((uint32_t)wave) * kWave >= a.s)
                continue;
            uint64_t r[N];
            int64_t e[N];
#pragma unroll
            for (int x = 0; x < N; ++x)
                r[x] = bounded64(draw64(rk, (uint32_t)((q + x) * kDrawThreads + tid)), W);
            find_entries<N>(a, d, top, r, e);
#pragma unroll
            for (int x = 0; x < N; ++x)
                key[q + x] = (q + x) * kDrawThreads + tid < a.s ? (uint32_t)a.p_col[e[x]] : kEmptySlot;
        }
    } else { // hardly any P at all, or an empty aggregated neighbourhood, which samples nothing
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const uint32_t j = (uint32_t)(q * kDrawThreads + tid);
            key[q] = kEmptySlot;
            if (j < (uint32_t)a.s && d.C > 0) {
                const uint64_t r = bounded64(draw64(rk, j), W);
                key[q] = (uint32_t)a.p_col[walk_entries(a, d, r)];
            }
        }
    }
    int turn = 0;
    sort_step<PER, 2, 1>(key, a.s, ex, turn);
    // the first of every run of equal columns stays
    uint32_t *sorted = ex + turn * PER * kDrawThreads;
#pragma unroll
    for (int q = 0; q < PER; ++q)
        sorted[q * kDrawThreads + tid] = key[q];
    __syncthreads();
    uint64_t heads[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int at = q * kDrawThreads + tid;
        heads[q] = __ballot(key[q] != kEmptySlot && (at == 0 || sorted[at > 0 ? at - 1 : 0] != key[q]));
        if (lane == 0)
            heads_of[at / kWave] = (uint32_t)__popcll(heads[q]);
    }
    __syncthreads();
    const uint32_t upto = wave_inclusive_scan_dpp(lane < PER * kDrawThreads / kWave ? heads_of[lane] : 0u);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)upto, kWave - 1);
    int32_t *__restrict__ out = PLACE ? a.col_vertex + place(total) : a.sel_tmp + (int64_t)i * a.s;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const uint32_t before = (uint32_t)__builtin_amdgcn_readlane((int)upto, q * (kDrawThreads / kWave) + (int)scalar((uint32_t)wave)) -
                                (uint32_t)__popcll(heads[q]);
        if ((heads[q] >> lane) & 1ull)
            out[before + bits_below(heads[q])] = (int32_t)key[q];
    }
    if (!PLACE && tid == 0)
        a.mb_count[i] = total;
}

__global__ __launch_bounds__(256) void ldw_sel_copy_kernel(LwHop a)
{
    if (a.giveup && *a.giveup)
        return;
    const int i = blockIdx.x;
    const int64_t c0 = a.mb_coloff[i], cnt = a.mb_coloff[i + 1] - c0;
    for (int64_t j = threadIdx.x; j < cnt; j += 256)
        a.col_vertex[c0 + j] = a.sel_tmp[(int64_t)i * a.s + j];
}

// ---------------------------------------------------------------------------------------------
// EXTRACT: blockIdx.y = minibatch; the workgroups of a minibatch share its tiles wave by wave
// ---------------------------------------------------------------------------------------------
// Hash of a column: its leading bits are a word of the filter (2^17 bits, 16 KB; 2^16 above 2048 sampled columns, so that two
// workgroups fit a compute unit) and one bit in it, five bits further down another one (with one bit 1.5 % of the neighbours passed,
// 2048 columns sampled, with two 0.25); its low ones are the place in the table (load factor <= 1/2).
// (A product of the last 24 bits is one step of the vector unit, of all 32 it is four; ids that differ further up only share a place.)
__device__ inline uint32_t ldw_hash(uint32_t v) { return (v & 0xFFFFFFu) * 0x9E3779u; }
__device__ inline uint32_t ldw_slot(uint32_t v, int32_t slots) { return (ldw_hash(v) >> 15) & (uint32_t)(slots - 1); }
struct FilterPlace {
    uint32_t word, bit, bit2;
};
__device__ inline FilterPlace ldw_filter(uint32_t hash, int filter_bits)
{
    return {hash >> (37 - filter_bits), (hash >> (32 - filter_bits)) & 31u, (hash >> (27 - filter_bits)) & 31u};
}

// A wave takes the positions of its tile 512 at a time, whatever rows they lie in: a row list of 64 rows at a time is held
// across the lanes, and where it matters (a step with more than one row) the row of a position follows from counting row
// starts up to it, as in the accumulation.  Going row by row instead left a wave with one short row's few lines in flight
// (two trips to memory of 2 us each per row: 75 k neighbours in rows of 49 took 55 us, 15 us so).
// Two workgroups per compute unit leave 64 registers.  The tile, its rows and what else a wave's lanes have in common are scalar;
// in every lane they cost 12 registers more, which went to memory and back (0.6 of 2.6 GB on 64 x 1024 seeds of 8.7 M vertices; 32 x
// 512 seeds, 3 layers of 512 of 2.4 M vertices: 86 us with, 69 us without).
// 64 x 1024 seeds of 8.7 M vertices, 237 M neighbours in a hop: 247 us with one bit of the filter per column, 221 with two; without
// whatever follows the filter it is 195 (4.9 TB/s), and a shorter filter step alone (29 -> 17 instructions per neighbour and lane) changed
// nothing.
struct ExtWave {
    int64_t shift[kWave];     // by rank among the list's rows with neighbours: A_col index of tile position 0 if it lay in the row
    uint32_t starts[kStreamUnroll * 2]; // one bit per position of a step: a row starts there
    uint32_t queue[2 * kWave];          // neighbours that passed the filter, in order
    uint16_t begin[kWave];    // by rank: where the row's piece begins in the tile
    uint16_t kept[kWave];     // by rank: neighbours of the piece found among the sampled columns
    uint8_t queue_rank[2 * kWave];
};

__global__ __launch_bounds__(kExtThreads, 8) void ldw_extract_kernel(LwHop a, int32_t slots, int filter_bits)
{
    extern __shared__ int64_t ext_lds[];
    ExtWave *waves = reinterpret_cast<ExtWave *>(ext_lds);
    uint32_t *maybe = reinterpret_cast<uint32_t *>(waves + kExtWaves); // the filter: ldw_filter's bits of the sampled columns
    uint32_t *hkey = maybe + (1 << filter_bits) / 32;                  // [slots]
    uint16_t *hval = reinterpret_cast<uint16_t *>(hkey + slots);       // [slots]
    if (a.giveup && *a.giveup)
        return;
    const int i = blockIdx.y, tid = threadIdx.x, lane = tid & (kWave - 1);
    const uint32_t wave = scalar((uint32_t)tid / kWave); // what is the same in a wave's lanes lies in scalar registers
    ExtWave &me = waves[wave];
    const int64_t c0 = a.mb_coloff[i];
    const int32_t ns = (int32_t)(a.mb_coloff[i + 1] - c0);
    const int64_t x0 = a.mb_gtileoff[i], ntiles = scalar(a.mb_gtileoff[i + 1] - x0);
    if (ns == 0 || (int64_t)blockIdx.x * kExtWaves >= ntiles)
        return; // nothing sampled: every row stays empty (the counters start at zero)
    for (int x = tid; x < slots; x += kExtThreads)
        hkey[x] = kEmptySlot;
    for (int x = tid; x < (1 << filter_bits) / 32; x += kExtThreads)
        maybe[x] = 0;
    __syncthreads();
    for (int j = tid; j < ns; j += kExtThreads) {
        const uint32_t v = (uint32_t)a.col_vertex[c0 + j];
        const FilterPlace f = ldw_filter(ldw_hash(v), filter_bits);
        atomicOr(&maybe[f.word], 1u << f.bit | 1u << f.bit2);
        uint32_t slot = ldw_slot(v, slots);
        while (atomicCAS(&hkey[slot], kEmptySlot, v) != kEmptySlot)
            slot = (slot + 1) & (uint32_t)(slots - 1);
        hval[slot] = (uint16_t)j;
    }
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1ull, below_incl = below | (1ull << lane);
    unsigned long long *rowcnt = reinterpret_cast<unsigned long long *>(a.out_rowptr);
    const int64_t nrows = a.mb_rowoff[a.k];
    // tiles cost very different amounts: the minibatch's tiles go to
    // whichever of its waves is free, off a shared counter, until none is left
    // A wave's first tile is its own number among the minibatch's waves; the counter hands out the tiles after
    // those.  The next tile is asked for before the current one is worked on, so that the answer (a trip to the
    // counter's home in memory, shared by all waves of the minibatch) is there when it is needed.  (Additions to one memory
    // line follow one another at about 8 ns each, so every counter has a line of its own, and waves that are at least as
    // many as tiles do not ask: 32 x 512, 7.6 M neighbours: 62 us when the counters shared lines, 27 so.)
    const int64_t nwaves = (int64_t)gridDim.x * kExtWaves;
    const int64_t g_first = scalar(a.mb_goff[i]), g_end = scalar(a.mb_goff[i + 1]);
    int64_t t = (int64_t)blockIdx.x * kExtWaves + wave;
    while (t < ntiles) {
        int64_t t_next = ntiles;
        if (lane == 0 && nwaves < ntiles)
            t_next = nwaves + (int64_t)atomicAdd(a.tile_queue + i * kQueueStride, 1ull);
        const int64_t g0 = g_first + t * a.tile;
        const int32_t len = (int32_t)(min(g0 + a.tile, g_end) - g0); // positions 0 .. len of the tile
        int64_t rw = scalar(a.tile_row[x0 + t]); // first row of the list
        int32_t p = 0;
        while (p < len) {
            const int64_t start = a.gather_off[min(rw + lane, nrows)], stop = a.gather_off[min(rw + lane + 1, nrows)];
            const bool row = stop > start; // with neighbours
            // in the tile; rows of other tiles are clamped to its ends
            const int32_t rs = (int32_t)max<int64_t>(min<int64_t>(start - g0, len), -1);
            const int32_t list_end = (int32_t)min<int64_t>(lane_value(stop, kWave - 1) - g0, len);
            const bool fresh = start >= g0, in_tile = row && start - g0 < len; // the piece is the row's first; there is one
            const int rank = __popcll(__ballot(row) & below);
            __builtin_amdgcn_wave_barrier();
            if (row) {
                me.shift[rank] = a.row_beg[rw + lane] - start + g0;
                me.begin[rank] = (uint16_t)max(rs, 0);
            }
            me.kept[lane] = 0;
            __builtin_amdgcn_wave_barrier();
            uint32_t qn = 0; // neighbours waiting in the wave's queue (the same in every lane)
            // looks the first n <= 64 queued neighbours up in the table, appends the local columns of those found
            // to their pieces' output in queue order, and moves the rest of the queue down
            auto drain = [&](uint32_t n) {
                __builtin_amdgcn_wave_barrier();
                const bool mine = (uint32_t)lane < n;
                const uint32_t val = mine ? me.queue[lane] : kEmptySlot;
                const int rk = mine ? (int)me.queue_rank[lane] : -1;
                int32_t local = -1;
                if (mine) {
                    uint32_t slot = ldw_slot(val, slots);
                    uint32_t kx;
                    while ((kx = hkey[slot]) != kEmptySlot) {
                        if (kx == val) {
                            local = hval[slot];
                            break;
                        }
                        slot = (slot + 1) & (uint32_t)(slots - 1);
                    }
                }
                const uint64_t found = __ballot(local >= 0);
                if (found) {
                    const int prev = __shfl_up(rk, 1, kWave), next = __shfl_down(rk, 1, kWave);
                    const uint64_t firsts = __ballot(mine && (lane == 0 || prev != rk)); // first queued one of every row
                    const uint64_t same = below & ~((1ull << (63 - __clzll((long long)(firsts & below_incl)))) - 1ull); // before this one, same row
                    const uint32_t at = mine ? me.kept[rk] + (uint32_t)__popcll(found & same) : 0u;
                    if (local >= 0)
                        a.xtmp[g0 + me.begin[rk] + at] = local; // the kept neighbours of a piece start where the piece starts
                    __builtin_amdgcn_wave_barrier();
                    if (mine && ((uint32_t)lane == n - 1u || next != rk)) // last queued one of its row
                        me.kept[rk] = (uint16_t)(at + (local >= 0 ? 1u : 0u));
                }
                const uint32_t rest = qn - n;
                const bool move = (uint32_t)lane < rest;
                const uint32_t moved = move ? me.queue[kWave + lane] : 0u;
                const uint8_t moved_rank = move ? me.queue_rank[kWave + lane] : 0;
                __builtin_amdgcn_wave_barrier();
                if (move) {
                    me.queue[lane] = moved;
                    me.queue_rank[lane] = moved_rank;
                }
                qn = rest;
                __builtin_amdgcn_wave_barrier();
            };
            for (; p < list_end; p += kStreamUnroll * kWave) {
                const int32_t n = min(list_end - p, kStreamUnroll * kWave);
                int rank0 = __popcll(__ballot(row && rs <= p)) - 1; // row of position p
                const bool inside = row && rs > p && rs < p + n;
                const bool one = __ballot(inside) == 0; // one row
                const int32_t left = n - lane;
                uint32_t v[kStreamUnroll];
                uint32_t ranks[kStreamUnroll / 4] = {}; // 8 bits each
                if (one) {
                    const int32_t *__restrict__ from = a.A_col + (scalar(me.shift[rank0]) + p);
                    if (n == kStreamUnroll * kWave) {
#pragma unroll
                        for (int u = 0; u < kStreamUnroll; ++u)
                            v[u] = (uint32_t)from[lane + u * kWave];
                    } else {
#pragma unroll
                        for (int u = 0; u < kStreamUnroll; ++u) {
                            v[u] = 0;
                            if (left > u * kWave)
                                v[u] = (uint32_t)from[lane + u * kWave];
                        }
                    }
                } else {
                    __builtin_amdgcn_wave_barrier();
                    if (lane < 2 * kStreamUnroll)
                        me.starts[lane] = 0;
                    __builtin_amdgcn_wave_barrier();
                    if (inside)
                        atomicOr(&me.starts[(rs - p) >> 5], 1u << ((rs - p) & 31));
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int u = 0; u < kStreamUnroll; ++u) {
                        const uint64_t m = reinterpret_cast<const uint64_t *>(me.starts)[u];
                        const int rk = rank0 + __popcll(m & below_incl);
                        rank0 += __popcll(m);
                        v[u] = 0;
                        if (left > u * kWave)
                            v[u] = (uint32_t)a.A_col[me.shift[rk] + (p + lane + u * kWave)];
                        ranks[u / 4] |= (uint32_t)rk << (8 * (u % 4));
                    }
                }
                // almost no neighbour is a sampled column: two bits of a word answer "certainly not" for
                // nearly all of them with a single LDS read each (all of a step's reads in flight together).
                // The few that pass are queued in row order; the table is searched a full wave of them at a
                // time (and at the end of the row list), not step by step
                uint32_t word[kStreamUnroll];
#pragma unroll
                for (int u = 0; u < kStreamUnroll; ++u)
                    word[u] = maybe[ldw_filter(ldw_hash(v[u]), filter_bits).word];
#pragma unroll
                for (int u = 0; u < kStreamUnroll; ++u) {
                    const int valid = n - u * kWave; // lanes
                    const FilterPlace f = ldw_filter(ldw_hash(v[u]), filter_bits);
                    const uint64_t pm = __ballot(((word[u] >> f.bit) & (word[u] >> f.bit2) & 1u) != 0u) &
                                        (valid >= kWave ? ~0ull : valid > 0 ? (1ull << valid) - 1ull : 0ull);
                    if (pm == 0)
                        continue;
                    if (__builtin_amdgcn_inverse_ballot_w64(pm)) {
                        const uint32_t at = qn + bits_below(pm);
                        me.queue[at] = v[u];
                        me.queue_rank[at] = (uint8_t)(one ? (uint32_t)rank0 : ranks[u / 4] >> (8 * (u % 4)));
                    }
                    qn += __popcll(pm);
                    if (qn >= (uint32_t)kWave)
                        drain(kWave);
                }
            }
            p = list_end;
            while (qn)
                drain(qn < (uint32_t)kWave ? qn : (uint32_t)kWave);
            if (in_tile) { // the pieces of the list's rows in this tile are done
                const uint32_t kept = me.kept[rank];
                const int64_t r = rw + lane;
                if (fresh)
                    a.first_cnt[r] = kept; // the piece a row starts with
                else
                    a.tile_cnt[x0 + t] = kept; // the piece a tile starts with, of a row begun earlier
                if (kept)
                    atomicAdd(&rowcnt[r], (unsigned long long)kept);
            }
            rw += kWave;
        }
        t = lane_value(t_next, 0);
    }
}

// rows to their place, piece by piece: 16 lanes per row
__global__ __launch_bounds__(256) void ldw_extract_copy_kernel(LwHop a)
{
    const int64_t R = a.mb_rowoff[a.k];
    if (a.giveup) {
        if (*a.giveup)
            return;
        if (a.out_rowptr[R] > a.col_cap) { // the kept neighbours do not fit what was provided
            if (blockIdx.x == 0 && threadIdx.x == 0)
                *a.giveup = 1;
            return;
        }
    }
    const int sub = threadIdx.x & 15;
    const int64_t groups = (int64_t)gridDim.x * 16;
    for (int64_t r = (int64_t)blockIdx.x * 16 + threadIdx.x / 16; r < R; r += groups) {
        int64_t o = a.out_rowptr[r];
        const int64_t total = a.out_rowptr[r + 1] - o;
        if (total == 0)
            continue;
        const int i = a.row_mb[r];
        const int64_t rs = a.gather_off[r], re = a.gather_off[r + 1];
        const int64_t gm = a.mb_goff[i], xm = a.mb_gtileoff[i];
        int64_t g = rs;
        int64_t cnt = a.first_cnt[r];
        int64_t t = (rs - gm) / a.tile;
        while (true) {
            for (int64_t j = sub; j < cnt; j += 16)
                a.out_col[o + j] = a.xtmp[g + j];
            o += cnt;
            ++t;
            g = gm + t * a.tile;
            if (g >= re)
                break;
            cnt = a.tile_cnt[xm + t];
        }
    }
}

// The scan of the rows' counts and the copy in one launch: 256 rows per workgroup, the rows before summed up by sum_before,
// then one entry per lane and step, whose row is found in the offsets in LDS.  Chains of trips to memory: what leads to a row's
// later pieces is fetched before the sum of the rows before, not after it (three layers of 32 x 512 seeds: 43 -> 37 us).
template <bool PUBLISH>
__device__ inline void extract_place(const LwHop &a, const Lookback &lb, int64_t *nnz_out, const PublishArgs &p)
{
    auto put = [](auto *p, auto v) {
        if (PUBLISH)
            store_through(p, v);
        else
            *p = v;
    };
    __shared__ int64_t smem[kLwRows / kWave];
    __shared__ uint32_t number_s;
    __shared__ int64_t gather_l[kLwRows], tile_l[kLwRows], pos_l[kLwRows]; // of a row: first kept neighbour, tile, that tile's first position
    __shared__ uint32_t off_l[kLwRows + 1], first_l[kLwRows];
    __shared__ int32_t up_s; // the flag as this workgroup sees it: it may go up meanwhile
    const int tid = threadIdx.x;
    if (tid == 0)
        up_s = a.giveup ? *a.giveup : 0;
    const uint32_t t = scalar(take_number(lb, &number_s));
    const int64_t R = uniform_load(a.mb_rowoff + a.k);
    const int64_t r0 = (int64_t)t * kLwRows, r = r0 + tid;
    if (t > 0 && r0 >= R)
        return;
    const int shift = __ffs(a.tile) - 1;
    int64_t cnt = 0, g = 0, gm = 0, xm = 0;
    int i = -1;
    if (!up_s && r < R) {
        i = a.row_mb[r];
        cnt = a.out_rowptr[r];
        g = a.gather_off[r];
        first_l[tid] = a.first_cnt[r];
        gm = a.mb_goff[i];
        xm = a.mb_gtileoff[i];
    }
    int64_t total;
    const int64_t ex = block_exclusive_scan<int64_t, kLwRows>(cnt, smem, total);
    off_l[tid] = (uint32_t)ex; // < 2^32: at most 256 rows of at most 4096 entries
    if (tid == 0)
        off_l[kLwRows] = (uint32_t)total;
    gather_l[tid] = g;
    tile_l[tid] = xm + ((g - gm) >> shift);
    pos_l[tid] = gm + ((g - gm) >> shift << shift);
    const int64_t before = sum_before<kLwRows>(lb, t, total, smem);
    int64_t *host_off = PUBLISH && p.off ? p.off + ((int64_t)(p.L - 1) * 3 + 1) * (a.k + 1) : nullptr; // first entries of the minibatches
    if (r < R) {
        put(a.out_rowptr + r, before + ex);
        for (; host_off && i >= 0 && a.mb_rowoff[i] == r; --i) // (and of those without rows before it)
            put(host_off + i, before + ex);
    }
    if (r0 + kLwRows >= R && tid == 0) {
        put(a.out_rowptr + R, before + total);
        put(nnz_out, before + total);
        if (PUBLISH)
            put(p.host + (nnz_out - p.scalars), before + total);
        for (i = a.k; host_off && i >= 0 && a.mb_rowoff[i] == R; --i)
            put(host_off + i, before + total);
    }
    if (PUBLISH && t == 0)
        publish_before<kLwRows>(p, nnz_out);
    if (a.giveup && before + total > a.col_cap) { // the kept neighbours do not fit what was provided
        if (tid == 0) {
            put(a.giveup, 1);
            if (PUBLISH)
                put(reinterpret_cast<int32_t *>(p.host + kRaisedSlot), 1);
        }
        return;
    }
    constexpr int kEach = 4; // entries per thread whose places are looked up before any of them is stored
    for (uint32_t x0 = 0; x0 < (uint32_t)total; x0 += kEach * kLwRows) {
        const uint32_t e0 = x0 + tid;
        int64_t from[kEach];
#pragma unroll
        for (int u = 0; u < kEach; ++u) {
            if (u && x0 + u * kLwRows >= (uint32_t)total) { // (no entry for any lane)
                from[u] = from[0];
                continue;
            }
            const uint32_t e = min(e0 + u * kLwRows, (uint32_t)total - 1u);
            int lo = 0; // last row whose entries begin at or before e: rows without entries share their begin
#pragma unroll
            for (int step = kLwRows / 2; step > 0; step /= 2)
                lo += off_l[lo + step] <= e ? step : 0;
            uint32_t x = e - off_l[lo], piece = first_l[lo];
            from[u] = gather_l[lo];
            if (x >= piece) { // in a later piece of the row: one per tile that it reaches into
                int32_t tile = 0; // after the row's first
                const uint32_t *__restrict__ counts = a.tile_cnt + tile_l[lo] + 1;
                do {
                    const U32x4_a4 c0 = *reinterpret_cast<const U32x4_a4 *>(counts + tile), c1 = *reinterpret_cast<const U32x4_a4 *>(counts + tile + 4);
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        const bool later = x >= piece;
                        x -= later ? piece : 0u;
                        piece = later ? (q < 4 ? c0[q % 4] : c1[q % 4]) : piece;
                        tile += later ? 1 : 0;
                    }
                } while (x >= piece);
                from[u] = pos_l[lo] + ((int64_t)tile << shift);
            }
            from[u] += x;
        }
        int32_t column[kEach];
#pragma unroll
        for (int u = 0; u < kEach; ++u)
            column[u] = a.xtmp[from[u]];
#pragma unroll
        for (int u = 0; u < kEach; ++u)
            if (e0 + u * kLwRows < (uint32_t)total)
                put(a.out_col + before + e0 + u * kLwRows, column[u]);
    }
}

// PUBLISH: the call's last launch, which leaves the sizes for the host as well
template <bool PUBLISH>
__global__ __launch_bounds__(kLwRows) void ldw_extract_place_kernel(LwHop a, Lookback lb, int64_t *nnz_out, PublishArgs p)
{
    extract_place<PUBLISH>(a, lb, nnz_out, p);
    if (PUBLISH)
        announce_through(p, gridDim.x);
}

// ---------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------
static void launch_ldw_tiles(const Launch &L, const LwHop &a)
{
    hipLaunchKernelGGL(ldw_plan_kernel, dim3(1), dim3(1024), 0, L.stream, a);
    hipLaunchKernelGGL(ldw_tile_rows_kernel, dim3(grid_for(L, (a.tiles_bound + 255) / 256, 8)), dim3(256), 0, L.stream, a);
}

bool ldw_fused(const LwHop &a) { return a.index && a.k < kPlanMb && (a.rows_bound + kLwRows - 1) / kLwRows <= kMostLookback; }

int launch_ldw_rows(const Launch &L, const LwHop &hop, const Lookback &lb, int64_t *gathered_out, uint32_t *workgroups)
{
    LwHop a = hop;
    const int64_t tiles = (a.rows_bound + kLwRows - 1) / kLwRows;
    if (tiles > kMostLookback)
        return -1;
    *workgroups = (uint32_t)tiles;
    int64_t more = a.seeds ? a.k : 0;
    size_t lds = 0;
    if (ldw_fused(a)) {
        const BoundsPieces pieces = bounds_pieces(L, a);
        a.bounds_width = pieces.width;
        more += grid_for(L, pieces.tiles, 8);
        lds = pieces.lds;
    }
    if (a.seeds)
        lds = std::max(lds, (size_t)a.seed_slots * sizeof(uint32_t));
    hipLaunchKernelGGL(ldw_rows_kernel, dim3((unsigned)(tiles + more)), dim3(kLwRows), lds, L.stream, a, lb, gathered_out, (int)tiles);
    return 0;
}

void launch_ldw_bounds(const Launch &L, const LwHop &hop)
{
    LwHop a = hop;
    const BoundsPieces pieces = bounds_pieces(L, a);
    a.bounds_width = pieces.width;
    launch_ldw_tiles(L, a);
    if (!a.index)
        hipLaunchKernelGGL(ldw_bounds_kernel, dim3(grid_for(L, (a.tiles_bound + 3) / 4, 8)), dim3(256), 0, L.stream, a);
    hipLaunchKernelGGL(ldw_bounds_transpose_kernel, dim3(grid_for(L, pieces.tiles, 8)), dim3(256), pieces.lds, L.stream, a);
}

void launch_ldw_index(const Launch &L, const LwHop &a)
{
    launch_ldw_tiles(L, a);
    hipLaunchKernelGGL(ldw_bounds_kernel, dim3(grid_for(L, (a.tiles_bound + 3) / 4, 8)), dim3(256), 0, L.stream, a);
}

template <bool NARROW, class Hop>
static int launch_accumulate(const Launch &L, const LwHop &a)
{
    void (*const kernels[2])(Hop) = {ldw_accumulate_kernel<false, NARROW>, ldw_accumulate_kernel<true, NARROW>};
    hipLaunchKernelGGL(kernels[a.squared ? 1 : 0], dim3(grid_for(L, (int64_t)a.k * a.nwin, NARROW ? 2 : 1)), dim3(kAccThreads<NARROW>),
                       0, L.stream, Hop{a});
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Counters of 8 bits where there are pairs for two workgroups per compute unit and few of them will be counted three times.
// `most`: the largest counter that is to be expected, a number that is off by up to 2 either way.  Whole calls of two layers, 16 and
// 8 bits: 266 pairs, 40 expected: 144 and 133 us; 320, 244: 234 and 208; 1064, 223: 279 and 268; 532, 462 (2 pairs overflow): 256 and
// 255; 920, 318 (12 overflow): 437 and 453; 532, 887 (92 overflow): 370 and 407.  With many pairs for every workgroup the few that
// overflow cost less: three layers, 8512 pairs, 325 expected (35 overflow): 3000 and 2820.
//
// Masks from kMaskEntries of a part on average on: below, the longer code costs 2 or 3 % of the accumulation and the copy gains nothing.  Calls of
// two layers, 64 minibatches, without and with them (entries a part in the second hop): 137 863 and 870 us, 151 226 and 228, 183 535 and 540, 246
// level, 268 level, 319 673 and 650, 439 342 and 338, 537 943 and 865.  Nor where few pairs' entries stay in the caches until the copy has read
// them, which is made for short parts.
int launch_ldw_accumulate(const Launch &L, LwHop &a, double most)
{
    const int64_t pairs = (int64_t)a.k * a.nwin;
    const bool narrow = pairs > L.num_cu && most <= (pairs >= 8 * L.num_cu ? 384.0 : 256.0);
    a.p_masks = narrow && !a.place_pairs && a.p_tune >= kMaskEntries * kWinParts * pairs ? 1 : 0;
    if (!narrow)
        return launch_accumulate<false, LwHop>(L, a);
    return a.p_masks ? launch_accumulate<true, LwMasks>(L, a) : launch_accumulate<true, LwHop>(L, a);
}

bool ldw_may_place(const LwHop &a) { return ldw_fused(a) && (int64_t)a.k * a.nwin <= kMostPlacedPairs; }

void launch_ldw_win_scan(const Launch &L, const LwHop &a, int64_t *pnnz_out)
{
    const int planners = ldw_fused(a) ? grid_for(L, (a.rows_bound + 4 * kScanThreads - 1) / (4 * kScanThreads), 1) : 0;
    hipLaunchKernelGGL(ldw_win_scan_kernel, dim3(a.k + planners), dim3(kScanThreads), 0, L.stream, a, pnnz_out);
}

template <class Hop>
static void launch_copy_parts(const Launch &L, const LwHop &a, int64_t workgroups)
{
    void (*const kernels[2][2])(Hop) = {{ldw_p_copy_kernel<false, false>, ldw_p_copy_kernel<false, true>},
                                        {ldw_p_copy_kernel<true, false>, ldw_p_copy_kernel<true, true>}};
    hipLaunchKernelGGL(kernels[a.squared ? 1 : 0][a.p_past ? 1 : 0], dim3((unsigned)workgroups), dim3(256), 0, L.stream, Hop{a});
}

void launch_ldw_p_copy(const Launch &L, const LwHop &a, int64_t *pnnz_out)
{
    if (a.place_pairs) {
        void (*const kernels[2][2])(LwHop, int, int64_t *) = {{ldw_p_place_kernel<false, 1024>, ldw_p_place_kernel<false, 256>},
                                                              {ldw_p_place_kernel<true, 1024>, ldw_p_place_kernel<true, 256>}};
        const int64_t pairs = (int64_t)a.k * a.nwin;
        const int nt = pairs <= 2 * L.num_cu ? 1024 : 256;
        const int planners = grid_for(L, (a.rows_bound + 4 * nt - 1) / (4 * nt), 1);
        hipLaunchKernelGGL(kernels[a.squared ? 1 : 0][nt == 1024 ? 0 : 1], dim3((unsigned)(pairs + planners)), dim3(nt), 0, L.stream, a,
                           planners, pnnz_out);
        return;
    }
    const int64_t workgroups = ((int64_t)a.k * a.nwin * kWinParts + 3) / 4;
    if (a.p_masks)
        launch_copy_parts<LwMasks>(L, a, std::min<int64_t>(workgroups, kMostCopying));
    else
        launch_copy_parts<LwHop>(L, a, grid_for(L, workgroups, 8));
}

int launch_ldw_draw(const Launch &L, const LwHop &a, const Lookback *lb, int64_t *ncols_out)
{
    void (*const kernels[3][3])(LwHop, Lookback, int64_t *, int) = {
        {ldw_draw_kernel<false, 1, false>, ldw_draw_kernel<false, 2, false>, ldw_draw_kernel<false, 4, false>},
        {ldw_draw_kernel<true, 1, false>, ldw_draw_kernel<true, 2, false>, ldw_draw_kernel<true, 4, false>},
        {ldw_draw_kernel<true, 1, true>, ldw_draw_kernel<true, 2, true>, ldw_draw_kernel<true, 4, true>}};
    static_assert(kMaxWinSampled <= 4 * kDrawThreads, "the sort is too short");
    const int per = a.s <= kDrawThreads ? 0 : a.s <= 2 * kDrawThreads ? 1 : 2;
    // 512 draws and more for each of several workgroups, as far as there are compute units: fewer gain less than the trip to memory and
    // back costs (32 minibatches, 512 draws, 256 for each of two: three hops 43 and 46 us).  Whole calls by one and by several, 2.4 M
    // vertices: 8 x 512 seeds, (1024, 1024) 159 and 156 us; 32 x 1024, (1024, 1024) 261 and 258; 128 x 512, (1024, 1024) 573 and 571;
    // 64 x 1024, (2048, 2048) 536 and 515; 3 x 512, (4096) 96 and 85.  Two for every compute unit: 123 for 100 us of three hops.
    const int parts = lb && a.k <= kMostSharedDraws ? std::max(1, std::min({8, a.s / 512, L.num_cu / a.k})) : 1;
    hipLaunchKernelGGL(kernels[parts > 1 ? 2 : lb ? 1 : 0][per], dim3(a.k * parts), dim3(kDrawThreads), 0, L.stream, a, lb ? *lb : Lookback{},
                       ncols_out, parts);
    return a.k * parts;
}

void launch_ldw_sel_copy(const Launch &L, const LwHop &a)
{
    hipLaunchKernelGGL(ldw_sel_copy_kernel, dim3(a.k), dim3(256), 0, L.stream, a);
}

void launch_ldw_extract(const Launch &L, const LwHop &a)
{
    int64_t per_mb = (L.num_cu * 2 + a.k - 1) / a.k; // workgroups per minibatch: about 2 per compute unit in all
    per_mb = std::min<int64_t>(per_mb, (a.tiles_bound + kExtWaves - 1) / kExtWaves); // never more than there are tiles
    per_mb = std::max<int64_t>(per_mb, 1);
    int32_t slots = 1024;
    while (slots < 2 * a.s)
        slots *= 2;
    const int filter_bits = a.s <= 2048 ? 17 : 16;
    const size_t lds = kExtWaves * sizeof(ExtWave) + (size_t)slots * 6 + ((size_t)1 << filter_bits) / 8;
    static bool attr_set = false;
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(ldw_extract_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                80 * 1024) != hipSuccess)
            (void)hipGetLastError(); // not required on every runtime
        attr_set = true;
    }
    hipLaunchKernelGGL(ldw_extract_kernel, dim3((unsigned)per_mb, a.k), dim3(kExtThreads), lds, L.stream, a, slots, filter_bits);
}

int launch_ldw_extract_place(const Launch &L, const LwHop &a, const Lookback &lb, int64_t *nnz_out, const PublishArgs *p, uint32_t *workgroups)
{
    const int64_t tiles = (a.rows_bound + kLwRows - 1) / kLwRows;
    if (tiles > kMostLookback)
        return -1;
    *workgroups = (uint32_t)tiles;
    if (p)
        hipLaunchKernelGGL(ldw_extract_place_kernel<true>, dim3((unsigned)tiles), dim3(kLwRows), 0, L.stream, a, lb, nnz_out, *p);
    else
        hipLaunchKernelGGL(ldw_extract_place_kernel<false>, dim3((unsigned)tiles), dim3(kLwRows), 0, L.stream, a, lb, nnz_out, PublishArgs{});
    return 0;
}

void launch_ldw_extract_copy(const Launch &L, const LwHop &a)
{
    hipLaunchKernelGGL(ldw_extract_copy_kernel, dim3(grid_for(L, (a.rows_bound + 15) / 16, 8)), dim3(256), 0, L.stream, a);
}

} // namespace bms
