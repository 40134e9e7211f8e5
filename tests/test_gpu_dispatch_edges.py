"""Sizes at which a call changes kernels, and the largest and smallest each kernel takes, against the oracle."""
import numpy as np
import pytest
import torch

from conftest import random_batches, random_csr, skewed_csr
from parity import assert_hops_equal

pytestmark = pytest.mark.gpu


def _check(rowptr, col, batches, fanouts, seed=3, calls=2, **variant):
    from oracle import bms_oracle as O
    from paper_2311_02909_amd import bms
    ref = O.sample_nodewise(rowptr, col, batches, fanouts, seed, 5, **variant)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = None
    for call in range(calls):   # the first call of a shape and a recycled one
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), fanouts, seed, mb_base=5, recycle=res, **variant)
        assert_hops_equal(res.hops(), ref, what="k=%d b=%d fanouts=%s %s call %d" % (*batches.shape, fanouts, variant, call))
    return res


@pytest.mark.parametrize("variant", [{}, {"replace": True}, {"union_dst": True}])
@pytest.mark.parametrize("s", [33, 63, 64, 65, 128, 129, 256, 257])
def test_wide_fanouts_at_the_limits_of_the_lists_in_registers(s, variant):
    rng = np.random.default_rng(500 + s)
    rowptr, col = skewed_csr(3000, 200_000, rng)
    _check(rowptr, col, random_batches(3000, 3, 70, rng), (s, 2), **variant)


# b * s around the 16384 entries that one workgroup sorts; the hop after it on the chip-wide path or in the same launch
@pytest.mark.parametrize("k,b,fanouts", [(2, 1024, (16,)), (2, 1025, (16, 2)), (3, 4096, (4, 3)), (1, 8192, (2, 2)),
                                         (2, 8193, (1, 1)), (5, 1, (1, 1, 1)), (1024, 3, (5, 4)), (1025, 3, (5, 4)),
                                         (4, 128, (8, 8, 2)), (4, 129, (8, 8, 2, 2)), (3, 512, (32, 2)), (3, 481, (17, 2))])
def test_hops_of_one_workgroup_per_minibatch(k, b, fanouts):
    rng = np.random.default_rng(b + k)
    n = 20_000
    rowptr, col = random_csr(n, 40.0, rng)
    _check(rowptr, col, random_batches(n, k, b, rng), fanouts)
    if b * (fanouts[0] + 1) <= 16400:
        _check(rowptr, col, random_batches(n, min(k, 8), b, rng), fanouts, union_dst=True, calls=1)
        _check(rowptr, col, random_batches(n, min(k, 8), b, rng), fanouts, replace=True, calls=1)


# hops whose tiles are sampled by dies (2 rows >= n, 8 minibatches and more; seven: in stacked order), the second one with minibatches
# of no, few and many tiles, which take different steps of the walk
@pytest.mark.parametrize("k", [7, 8, 9, 37])
@pytest.mark.parametrize("variant", [{}, {"replace": True}, {"union_dst": True}], ids=lambda v: "+".join(v))
def test_tiles_by_dies_with_minibatches_of_unequal_length(k, variant):
    rng = np.random.default_rng(900 + k)
    n, b = 20_000, 1500
    lists = [np.zeros(0, dtype=np.int64)] * n
    for v in range(2000, 11_000):      # many tiles
        lists[v] = np.unique(rng.integers(0, n, size=40))
    for v in range(11_000, n):         # two tiles
        lists[v] = np.unique(rng.integers(11_000, 11_300, size=40))
    rowptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    col = np.concatenate(lists).astype(np.int32)
    groups = [np.arange(2000, 11_000), np.arange(11_000, n), np.arange(2000), np.arange(2000, n)]
    batches = np.stack([rng.choice(groups[i % 4], size=b, replace=False) for i in range(k)]).astype(np.int32)
    _check(rowptr, col, batches, (14, 5), **variant)


# the same of hops whose entries are counted per segment (8 rows >= n, up to 128 segments): by dies after every tile, or, of more
# segments, in stacked order; the second call has more tiles than the first makes likely, and the third as many segments as the
# second had entries for: 128 and 129 of the larger graphs (independent draws 64 and 65)
@pytest.mark.parametrize("variant", [{}, {"union_dst": True}, {"replace": True}], ids=lambda v: "+".join(v))
@pytest.mark.parametrize("n,per_mb", [(60_000, 45_000), (128 * 32768, 16384 * 128), (128 * 32768 + 1, 16384 * 128)])
def test_tiles_by_dies_that_count_per_segment(n, per_mb, variant):
    from oracle import bms_oracle as O
    from paper_2311_02909_amd import bms
    rng = np.random.default_rng(n)
    k, b = 9, 1200
    first = 60 if n < 1_000_000 else 200            # the first hop's neighbours, so that the second has rows for every eighth vertex
    second = per_mb // (b * first) + 1
    few = second // 2 + 1                           # neighbours of what the first call reaches
    half = n // 2                                   # even vertices lead to one another, and so do odd ones
    lengths = np.full(n, second)
    lengths[::2] = few
    lengths[:2 * k * b:2], lengths[1:2 * k * b:2] = first // 2, first
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    row = np.repeat(np.arange(n), lengths)
    at = np.arange(len(row)) - rowptr[row]          # one neighbour out of each of as many stretches of its kind
    stretch = half // lengths[row]
    col = (2 * (at * stretch + rng.integers(0, 1 << 30, len(row)) % stretch) + row % 2).astype(np.int32)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    fanouts = (first, 8)
    res = None
    for call in range(3):
        batches = (2 * np.arange(k * b, dtype=np.int32) + (1 if call == 1 else 0)).reshape(k, b)
        ref = O.sample_nodewise(rowptr, col, batches, fanouts, 5, **variant)
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as profile:
            res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), fanouts, 5, extract="sort", recycle=res, **variant)
            torch.cuda.synchronize()
        assert_hops_equal(res.hops(), ref, what="call %d" % call)
        names = [e.name.split("(")[0] for e in profile.events()]
        sample = [x for x in names if "nw_sample_kernel<8," in x][-1]
        by_dies = "true>" in sample.split(",")[-1]
        assert 8 * res.sizes()[1][0] >= n and res.attempts() == 1
        # (segments by the entries that the call before had)
        assert by_dies == (n <= 128 * 32768 or call < 2 or "replace" in variant), sample
        # ... and the sampling kernel counted: no pass over the entries does
        after = names[len(names) - names[::-1].index(sample):]
        assert any("dd_split_kernel" in x for x in after) and not any("dd_count_kernel" in x for x in after), after


# ... and up to 27 MB of columns per tile of a minibatch: many minibatches whose rows fill one tile and part of a second
@pytest.mark.parametrize("more", [0, 1])
def test_tiles_by_dies_of_many_minibatches_with_few_rows(more):
    from oracle import bms_oracle as O
    from paper_2311_02909_amd import bms
    rng = np.random.default_rng(43)
    n, k, b, entries = 150_000, 72, 100, (27 << 20) // 4 + more
    lengths = np.full(n, entries // n)
    lengths[:entries - lengths.sum()] += 1
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    row = np.repeat(np.arange(n), lengths)
    stretch = n // lengths[row]
    col = ((np.arange(entries) - rowptr[row]) * stretch + rng.integers(0, 1 << 30, entries) % stretch).astype(np.int32)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = None
    for call in range(3):
        batches = random_batches(n, k, b, rng)
        ref = O.sample_nodewise(rowptr, col, batches, (5, 8), 5 + call)
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as profile:
            res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (5, 8), 5 + call, extract="sort", recycle=res)
            torch.cuda.synchronize()
        assert_hops_equal(res.hops(), ref, what="call %d" % call)
        assert res.sizes()[1][0] // k // 256 == 1 and 8 * res.sizes()[1][0] >= n
        sample = [e.name.split("(")[0] for e in profile.events() if "nw_sample_kernel<8," in e.name][-1]
        assert ("true>" in sample.split(",")[-1]) == (not more), (call, sample)


# tiles by dies in one round of what the chip holds at a time, in a second that is half empty (workgroups go on then), and in more
@pytest.mark.parametrize("variant", [{}, {"union_dst": True}], ids=lambda v: "+".join(v))
@pytest.mark.parametrize("k", [20, 30, 40])
def test_rounds_of_tiles_by_dies(k, variant):
    from oracle import bms_oracle as O
    from paper_2311_02909_amd import bms
    rng = np.random.default_rng(44)
    n, b = 20_000, 1000
    col = ((np.arange(n * 40) % 40) * (n // 40) + rng.integers(0, n // 40, n * 40)).astype(np.int32)
    rowptr = np.arange(0, n * 40 + 1, 40, dtype=np.int64)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = None
    for call in range(3):
        batches = random_batches(n, k, b, rng)
        ref = O.sample_nodewise(rowptr, col, batches, (30, 10), 5 + call, **variant)
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as profile:
            res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (30, 10), 5 + call, recycle=res, **variant)
            torch.cuda.synchronize()
        assert_hops_equal(res.hops(), ref, what="call %d" % call)
        sample = [e.name.split("(")[0] for e in profile.events() if "nw_sample_kernel<16," in e.name][-1]
        assert "true>" in sample.split(",")[-1], sample
        tiles = res.sizes()[1][0] // k // 256
        rounds = k * (tiles + tiles // 8 + 3) / (5 * torch.cuda.get_device_properties(0).multi_processor_count)
        assert (1.2 < rounds < 2) == (k == 30), rounds


# ids that crowd a part of the range: the second hop's segments are of unequal width, its entries are counted through their table, and
# its tiles are sampled in stacked order, also where there are rows for every vertex and few segments
@pytest.mark.parametrize("variant", [{}, {"union_dst": True}, {"replace": True}], ids=lambda v: "+".join(v))
def test_tiles_in_stacked_order_with_a_table_of_segments(variant):
    from oracle import bms_oracle as O
    from paper_2311_02909_amd import bms
    rng = np.random.default_rng(41)
    n, k, b = 60_000, 9, 1200
    lists = [np.unique(rng.integers(0, n, size=64)) for _ in range(k * b)]
    lists += [np.unique(np.concatenate([rng.integers(0, 900, size=36), rng.integers(0, n, size=4)])) for _ in range(n - k * b)]
    rowptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    col = np.concatenate(lists).astype(np.int32)
    batches = np.arange(k * b, dtype=np.int32).reshape(k, b)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = None
    for call in range(3):
        ref = O.sample_nodewise(rowptr, col, batches, (60, 8), 5 + call, **variant)
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as profile:
            res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (60, 8), 5 + call, extract="sort", recycle=res, **variant)
            torch.cuda.synchronize()
        assert_hops_equal(res.hops(), ref, what="call %d" % call)
        names = [e.name.split("(")[0] for e in profile.events()]
        sample = [x for x in names if "nw_sample_kernel<8," in x][-1]
        assert 2 * res.sizes()[1][0] >= n
        if call:        # the table is at hand
            assert res.attempts() == 1 and any("dd_split_kernel" in x and "true>" in x for x in names), names
            assert not any("dd_count_kernel" in x for x in names[names.index(sample):]), names
            assert "false>" in sample.split(",")[-1], sample


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 16384, 16385, 70_000, 3_000_000])
def test_one_workgroup_hops_over_vertex_ranges_and_hubs(n):
    # a few hubs that every row samples crowd one bucket of ids: the counting passes take over
    rng = np.random.default_rng(n)
    m = min(20 * n, 300_000)
    hubs = rng.integers(0, n, size=3)
    src = rng.integers(0, n, size=m)
    dst = np.where(rng.random(m) < 0.5, hubs[rng.integers(0, 3, size=m)], rng.integers(0, n, size=m))
    key = np.unique(src * n + dst)
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.add.at(rowptr, key // n + 1, 1)
    rowptr, col = np.cumsum(rowptr), (key % n).astype(np.int32)
    b = min(n, 300)
    for variant in ({}, {"union_dst": True}):
        _check(rowptr, col, random_batches(n, 3, b, rng, candidates=np.unique(key // n) if len(np.unique(key // n)) >= b else None),
               (6, 3), **variant)


def test_places_beyond_32_bits():
    # a closed set of vertices whose lists lie behind 2^32 entries: the kernels cannot stage their places in 32-bit words.
    # The entries before it are the lists of vertices that nothing leads to, so the oracle gets the graph without them.
    from oracle import bms_oracle as O
    from paper_2311_02909_amd import bms
    rng = np.random.default_rng(77)
    pad, m = 65536, 3000
    rowptr, col = skewed_csr(m, 90_000, rng)
    n = pad + m
    small_rowptr = np.concatenate([np.zeros(pad, dtype=np.int64), rowptr])
    small_col = (col + pad).astype(np.int32)
    big_rowptr = np.concatenate([np.arange(pad, dtype=np.int64) * pad, rowptr + pad * pad])
    big_col = torch.empty(pad * pad + len(col), dtype=torch.int32, device="cuda")
    big_col[:pad * pad].view(pad, pad)[:] = torch.arange(pad, dtype=torch.int32, device="cuda")
    big_col[pad * pad:] = torch.from_numpy(small_col).cuda()
    csr = bms.Csr(torch.from_numpy(big_rowptr).cuda(), big_col)
    candidates = np.arange(pad, n)
    for b, fanouts in ((64, (5, 5)), (700, (20, 10)), (300, (40, 30))):
        batches = random_batches(n, 3, b, rng, candidates=candidates)
        for variant in ({}, {"union_dst": True}, {"replace": True}):
            ref = O.sample_nodewise(small_rowptr, small_col, batches, fanouts, 9, **variant)
            got = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), fanouts, 9, **variant)
            assert_hops_equal(got.hops(), ref, what="b=%d fanouts=%s %s" % (b, fanouts, variant))


# EXTRACT by bitmaps of vertex ranges: quads of 128 ids, ranges of 1024 quads and more, tables of 4864; minibatches in groups of
# 8; up to 4 of them with their bits set by the sampling kernel, more by a kernel of their own
@pytest.mark.parametrize("n,b", [(1, 1), (127, 100), (129, 129), (131_073, 900), (622_592, 1400), (622_593, 1400), (1_300_001, 2600)])
def test_extract_by_vertex_ranges(n, b):
    rng = np.random.default_rng(n)
    rowptr, col = random_csr(n, min(14.0, n / 2), rng)
    for k, variant in ((4, {}), (5, {"union_dst": True}), (9, {}), (1, {"union_dst": True}), (16, {"replace": True})):
        _check(rowptr, col, random_batches(n, k, b, rng), (40, 2), **variant)
    if n > 100_000:  # the sampled ids of the rows in one launch, then ranges
        _check(rowptr, col, random_batches(n, 6, b, rng), (3, 13), union_dst=True)


# layer-wise: rows and minibatches up to which workgroups add up those before them (262144 and 1024), k from which the plan is a
# launch of its own (1024), table sizes of the extraction, lists of 64 rows in which most have no neighbours or one
@pytest.mark.parametrize("n,deg,k,b,s", [(3000, 6.0, 1024, 3, (4, 3)), (3000, 6.0, 1023, 3, (3,)), (3000, 6.0, 1025, 2, (3, 4)),
                                         (30_000, 4.0, 291, 900, (5, 7)), (30_000, 4.0, 293, 900, (5, 7)), (90_000, 0.8, 3, 5000, (2048, 60)),
                                         (90_000, 0.8, 2, 5000, (2049, 4096)), (70_000, 60.0, 2, 700, (4096, 513))])
def test_layerwise_limits(n, deg, k, b, s):
    from oracle import bms_oracle as O
    from paper_2311_02909_amd import bms
    rng = np.random.default_rng(n + k + b)
    rowptr, col = random_csr(n, deg, rng)
    batches = random_batches(n, k, b, rng)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    for squared in (False, True):
        ref = O.sample_ladies(rowptr, col, batches, s, 17, 5, squared)
        res = None
        for index in (True, True, False):
            res = bms.sample_ladies(csr, torch.from_numpy(batches).cuda(), s, 17, mb_base=5, squared=squared, recycle=res, index=index)
            assert_hops_equal(res.hops(), ref, with_p=True, what="k=%d b=%d s=%s squared=%s index=%s" % (k, b, s, squared, index))


# EXTRACT by bitmaps in LDS of id ranges: ids of a range in registers (10240) or read again, distinct ids that have room in LDS (10240)
# or leave one by one, ranges of a few ids and of 2^18; tiles of 8192 positions taken apart and put together again
@pytest.mark.parametrize("n,used,b,s", [(9000, 1.0, 4096, 2), (9000, 1.0, 4097, 4), (60_000, 1.0, 9000, 25), (400_000, 0.5, 20_000, 10),
                                        (800_000, 0.3, 20_000, 10), (2_000_000, 1.0, 3000, 6), (1_500_000, 1.0, 12_000, 12)])
def test_extract_by_bitmaps_of_id_ranges(n, used, b, s):
    from oracle import bms_oracle as O
    from paper_2311_02909_amd import bms
    rng = np.random.default_rng(n + b)
    rowptr = np.zeros(n + 1, dtype=np.int64)
    rows = rng.choice(n, size=b, replace=False)
    rowptr[rows + 1] = s + rng.integers(0, 3, size=b)
    rowptr = np.cumsum(rowptr)
    gaps = rng.integers(1, max(int(used * n) // (s + 3), 2), size=(b, s + 2))
    ids = np.minimum(np.cumsum(gaps, axis=1) - 1, n - 1)
    row = np.repeat(np.arange(n), np.diff(rowptr))
    slot = np.arange(len(row)) - rowptr[row]
    which = np.searchsorted(np.sort(rows), row)
    col = ids[which, slot].astype(np.int32)
    batches = np.stack([rng.permutation(rows) for _ in range(3)]).astype(np.int32)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    for variant in ({}, {"union_dst": True}, {"replace": True}):
        ref = O.sample_nodewise(rowptr, col, batches, (s,), 3, 5, **variant)
        res = None
        for call in range(2):
            res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (s,), 3, mb_base=5, recycle=res, extract="sort", **variant)
            assert_hops_equal(res.hops(), ref, what="n=%d b=%d s=%d %s call %d" % (n, b, s, variant, call))


# ... and the forms that few, many and large minibatches of such graphs take: bitmaps set by several workgroups and merged (parts 4 to
# 32) or by one, over ranges of 1024 to 5120 quads; look-ups of 8, 16, 32 and 56 ids per thread in 1, 3, 4, 6 and 8 tables
@pytest.mark.parametrize("n,k,b,s", [(300_000, 5, 1500, 150), (300_000, 64, 500, 100), (300_000, 64, 1500, 150), (600_000, 16, 1500, 150),
                                     (1_000_000, 70, 600, 60), (1_300_001, 24, 1500, 150), (2_450_000, 64, 500, 100),
                                     (3_700_000, 16, 2000, 300), (4_900_000, 6, 1500, 150)])
def test_forms_of_extract_by_vertex_ranges(n, k, b, s):
    from oracle import bms_oracle as O
    from paper_2311_02909_amd import bms
    rng = np.random.default_rng(n + k)
    rowptr = np.zeros(n + 1, dtype=np.int64)
    rows = np.sort(rng.choice(n, size=b + 7, replace=False))
    rowptr[rows + 1] = s + rng.integers(0, 3, size=b + 7)
    rowptr = np.cumsum(rowptr)
    steps = rng.integers(1, 2 * n // (s + 3), size=(b + 7, s + 2))   # of a row's list, over [0, n)
    ids = np.sort(np.cumsum(steps, axis=1) % (n - s - 2), axis=1) + np.arange(s + 2)   # strictly ascending
    row = np.repeat(np.arange(n), np.diff(rowptr))
    col = ids[np.searchsorted(rows, row), np.arange(len(row)) - rowptr[row]].astype(np.int32)
    batches = np.stack([rng.permutation(rows)[:b] for _ in range(k)]).astype(np.int32)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    for variant in ({}, {"union_dst": True}):
        ref = O.sample_nodewise(rowptr, col, batches, (s,), 3, 5, **variant)
        res = None
        for profile in (False, False, "as_run"):
            res = bms.sample_nodewise(csr, batches, (s,), 3, mb_base=5, recycle=res, profile=profile, **variant)
            assert_hops_equal(res.hops(), ref, what="n=%d k=%d b=%d s=%d %s" % (n, k, b, s, variant))
        assert "rg_mark" in {x for x, _, _ in res.stages()}


def _few_long_rows(n, b, s, rng):
    """A graph of n vertices of which b, spread over [0, n), have s random neighbours each; on the device."""
    from paper_2311_02909_amd import bms
    rows = np.sort(rng.choice(n, size=b, replace=False))
    degree = torch.zeros(n, dtype=torch.int64, device="cuda")
    degree[torch.from_numpy(rows).cuda()] = s
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(degree, 0, out=rowptr[1:])
    col = np.sort(rng.integers(0, n - s, size=(b, s)), axis=1) + np.arange(s)
    return bms.Csr(rowptr, torch.from_numpy(col.astype(np.int32).reshape(-1)).cuda()), rows


@pytest.mark.parametrize("n,k,by_bits", [(2_000_000, 4, True), (31_000_000, 3, True), (33_000_000, 3, False), (95_000_000, 1, True),
                                         (97_000_000, 1, False)])
def test_few_minibatches_of_large_graphs_go_by_segments(n, k, by_bits):
    # bitmaps in memory are cleared, counted and read as a whole: 96 million bits, in all minibatches, is where that ends
    from paper_2311_02909_amd import bms
    rng = np.random.default_rng(k)
    csr, rows = _few_long_rows(n, 1200, 60, rng)
    batches = torch.from_numpy(np.stack([rng.permutation(rows)[:1000] for _ in range(k)]).astype(np.int32)).cuda()
    got, by_segments = (bms.sample_nodewise(csr, batches, (50,), 3, profile="as_run", extract=x) for x in (None, "sort"))
    assert ("rg_count" in {x for x, _, _ in got.stages()}) == by_bits
    assert "dd_split" in {x for x, _, _ in by_segments.stages()}
    for a, b in zip(got.hops(), by_segments.hops()):
        assert torch.equal(a.rowptr, b.rowptr) and torch.equal(a.col, b.col) and torch.equal(a.col_vertex, b.col_vertex)
        assert torch.equal(a.mb_coloff, b.mb_coloff)


def test_bitmaps_of_vertex_ranges_stay_inside_the_scratch_limit():
    # few large minibatches have their ids marked by up to 32 workgroups with a bitmap each: only as many as the limit has room for
    from paper_2311_02909_amd import bms
    rng = np.random.default_rng(4)
    n, k = 300_000, 5
    csr, rows = _few_long_rows(n, 1600, 160, rng)
    batches = torch.from_numpy(np.stack([rng.permutation(rows)[:1500] for _ in range(k)]).astype(np.int32)).cuda()
    limit, ref = 6_000_000, None
    for scratch_limit in (limit, limit, 0):
        res = bms.sample_nodewise(csr, batches, (150,), 3, profile="as_run", scratch_limit=scratch_limit)
        assert "rg_mark" in {x for x, _, _ in res.stages()}
        assert (csr.held_bytes() <= limit) == (scratch_limit == limit), csr.held_bytes()
        got = [(h.rowptr.cpu(), h.col.cpu(), h.col_vertex.cpu(), h.mb_coloff.cpu()) for h in res.hops()]
        ref = ref or got
        for a, b in zip(got, ref):
            assert all(torch.equal(x, y) for x, y in zip(a, b))


def test_bitmaps_of_all_hops_are_allocated_before_the_first_one_runs():
    # hop 0 takes one bitmap per minibatch, hop 1 several: what the handle holds is looked at when the result's buffers are allocated
    from oracle import bms_oracle as O
    from paper_2311_02909_amd import bms
    rng = np.random.default_rng(21)
    rowptr, col = random_csr(300_000, 14.0, rng)
    batches = random_batches(300_000, 5, 1500, rng)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    held, allocator = [], bms.TorchAllocator()
    alloc = allocator.alloc

    def look(nbytes, ctx):
        held.append(csr.held_bytes())
        return alloc(nbytes, ctx)
    allocator.alloc = bms.ALLOC_FN(look)
    res = bms.sample_nodewise(csr, batches, (40, 40), 3, allocator=allocator)
    assert_hops_equal(res.hops(), O.sample_nodewise(rowptr, col, batches, (40, 40), 3), what="two hops by ranges")
    assert len(held) == 2 + 2 * 4   # seeds and their offsets, then per hop row and column offsets, columns and their vertices
    rows = res.hop(0).nnz           # the bound of hop 1's rows: 12 bytes each, and 8 per tile of 256
    assert held[-1] - held[5] <= 13 * rows + 4096, held
    parts = bms.sample_nodewise(csr, batches, (40, 40), 3, recycle=res, profile="as_run")
    assert {(x, h) for x, h, _ in parts.stages()} >= {("rg_mark", 0), ("rg_mark", 1)}


def _kernels(call):
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as profile:
        call()
        torch.cuda.synchronize()
    return [e.name for e in profile.events() if "nw_sample" in e.name]


@pytest.mark.parametrize("degree,b,s,wide", [(12.0, 1024, 64, True), (12.0, 400, 40, True), (100.0, 276, 48, False)])
def test_wide_fanouts_by_the_rows_there_are(degree, b, s, wide):
    # the second hop's rows are 54000, 21000 and 60000 where k b s bounds them by more than 65536: by waves, or by lanes for their
    # 3 million entries, in the first call and in recycled ones
    from oracle import bms_oracle as O
    from paper_2311_02909_amd import bms
    rng = np.random.default_rng(b)
    rowptr, col = random_csr(120_000, degree, rng)
    batches = random_batches(120_000, 5, b, rng)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    ref = O.sample_nodewise(rowptr, col, batches, (s, s), 3)
    res, names = None, []
    for call in range(3):
        def once():
            nonlocal res
            res = bms.sample_nodewise(csr, batches, (s, s), 3, recycle=res)
        names.append(_kernels(once))
        assert_hops_equal(res.hops(), ref, what="call %d" % call)
    rows, entries, _ = res.sizes()[1]
    assert len(batches) * b * s > 65536 > rows and (entries < 900_000) == wide, (rows, entries)
    assert all(len(x) == 2 and ("wide" in x[1]) == wide for x in names), names


def _segments(n, per_minibatch):
    """id ranges that EXTRACT by segments cuts a hop of so many entries per minibatch into"""
    dense = n <= 128 * (per_minibatch + 1)
    shift = 0
    while shift < (18 if dense else 31) and (2 << shift) * (per_minibatch + 1) <= (16384 if dense else 3000) * n:
        shift += 1
    return -(-n // (1 << shift))


# EXTRACT by segments: minibatches that begin anywhere in a memory line of 32 entries, of one tile of 8192 entries, a few more and a few
# less, of several tiles and of none; one segment, so that a tile is one run, some, and more than the 512 that a workgroup takes at a time
@pytest.mark.parametrize("variant", [{}, {"union_dst": True}], ids=lambda v: "+".join(v))
@pytest.mark.parametrize("n,b,base,segments", [(60_000, 40, 0, 1), (14_000_000, 130, 98_304, 54), (200_000_000, 1400, 1_310_720, 763)])
def test_tiles_of_the_cut_at_memory_lines(n, b, base, segments, variant):
    from oracle import bms_oracle as O
    from paper_2311_02909_amd import bms
    rng = np.random.default_rng(77)
    sizes = [8192, 1, 8161, 8160, 0, 8192, 8193, 8191 + 31, 8192 + 31, 16384 - 7, 33, 16384 + 1, 31, 24576]
    sizes = [base + size if size else 0 for size in (sizes if segments < 512 else sizes[:4])]
    assert _segments(n, sum(sizes) / len(sizes)) == segments
    rows = []
    for size in sizes:                  # the seeds of a minibatch have `size` neighbours together, all of them kept
        parts = np.full(b, size // b)
        parts[:size % b] += 1           # (one neighbour out of each of as many stretches of the ids)
        rows += [np.arange(p) * (n // max(p, 1)) + rng.integers(0, n // max(p, 1), p) for p in parts]
    rowptr = np.zeros(n + 1, dtype=np.int64)
    rowptr[1:len(rows) + 1] = np.cumsum([len(r) for r in rows])
    rowptr[len(rows) + 1:] = rowptr[len(rows)]
    col = np.concatenate(rows).astype(np.int32)
    batches = np.arange(len(rows), dtype=np.int32).reshape(len(sizes), b)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    ref = O.sample_nodewise(rowptr, col, batches, (1024,), 5, 0, **variant)
    res = None
    for call in range(2):
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (1024,), 5, extract="sort", recycle=res, **variant)
        assert_hops_equal(res.hops(), ref, what="call %d" % call)


# the cut starts a workgroup for every tile that the call before makes likely: a call of three times the entries has more
@pytest.mark.parametrize("n", [400_000, 20_000_000])    # segments by bitmaps, and by counting
def test_more_tiles_than_the_call_before(n):
    from oracle import bms_oracle as O
    from paper_2311_02909_amd import bms
    rng = np.random.default_rng(79)
    b, few, many = 2000, 30, 60 if n > 1_000_000 else 90    # (by counting, a segment takes twice what it is made for)
    lengths = np.zeros(n, dtype=np.int64)
    lengths[:2 * b], lengths[2 * b:4 * b] = few, many
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    col = np.concatenate([np.arange(x) * (n // x) + rng.integers(0, n // x, x) for x in lengths[:4 * b]]).astype(np.int32)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = None
    for call in range(3):
        batches = (np.arange(2 * b, dtype=np.int32) + (2 * b if call == 1 else 0)).reshape(2, b)
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (100,), 5, extract="sort", recycle=res)
        assert_hops_equal(res.hops(), O.sample_nodewise(rowptr, col, batches, (100,), 5), what="call %d" % call)
        assert res.attempts() == 1


def test_scratch_of_the_cut_goes_by_entries():
    # many minibatches of hardly any entries: scratch by what they hold, not by a tile each (16 KB)
    from oracle import bms_oracle as O
    from paper_2311_02909_amd import bms
    rng = np.random.default_rng(78)
    k = 20_000
    rowptr, col = random_csr(3000, 6.0, rng)
    batches = random_batches(3000, k, 2, rng)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    ref = O.sample_nodewise(rowptr, col, batches, (4, 3), 5)
    res = None
    for call in range(2):
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (4, 3), 5, extract="sort", recycle=res)
        assert_hops_equal(res.hops(), ref, what="call %d" % call)
    bound = 2 * k * 4 * 3           # entries of the second hop, at most
    assert csr.held_bytes() <= 64 * bound + 512 * k


# more tiles of rows than one workgroup scans (32768), a chunk of 4096 and one more or less of them
@pytest.mark.parametrize("k", [32768, 32769, 36864, 36865])
def test_scans_over_many_tiles(k):
    rng = np.random.default_rng(k)
    rowptr, col = random_csr(3000, 6.0, rng)
    _check(rowptr, col, random_batches(3000, k, 2, rng), (3, 2))
