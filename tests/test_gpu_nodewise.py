"""Parity of the HIP node-wise sampler with the CPU oracle (bit-exact), through the C ABI."""
import numpy as np
import pytest
import torch

from conftest import random_batches, random_csr, skewed_csr
from parity import assert_hops_equal

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mods():
    from oracle import bms_oracle as O
    from paper_2311_02909_amd import bms, synth
    assert torch.cuda.is_available()
    return O, bms, synth


def _run_both(mods, rowptr, col, batches, fanouts, seed, mb_base=0, device_csr=True):
    """Runs every EXTRACT kernel path of the library and compares each with the oracle."""
    O, bms, _ = mods
    rp, cl = torch.from_numpy(rowptr), torch.from_numpy(col)
    if device_csr:
        rp, cl = rp.cuda(), cl.cuda()
    csr = bms.Csr(rp, cl)
    ref = O.sample_nodewise(rowptr, col, batches, fanouts, seed, mb_base)
    for extract in ("sort", "buckets", "bitmap"):
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), fanouts, seed, mb_base=mb_base,
                                  extract=extract)
        assert_hops_equal(res.hops(), ref, what="extract=%s fanouts=%s seed=%d" % (extract, fanouts, seed))
    return csr, res, ref


def test_tiny_workload(mods):
    O, bms, synth = mods
    g, batches, w = synth.make_workload("tiny_sage")
    print("tiny_sage:", g.describe(), flush=True)
    _run_both(mods, g.rowptr.numpy(), g.col.numpy(), batches.numpy(), w["params"], synth.SAMPLING_SEED)


@pytest.mark.parametrize("fanouts", [(3,), (4, 4), (5, 5), (8, 3, 2), (15, 10, 5), (16, 2), (17, 3), (32, 2), (1, 1, 1)])
def test_random_graph_all_lane_capacities(mods, fanouts):
    # n and b chosen so that a minibatch spans several 256-row tiles with a ragged tail
    rng = np.random.default_rng(sum(fanouts))
    rowptr, col = random_csr(20000, 24.0, rng)
    batches = random_batches(20000, 5, 300, rng)
    _run_both(mods, rowptr, col, batches, fanouts, 7, mb_base=3)


@pytest.mark.parametrize("fanouts", [(33, 2), (40, 40), (200, 3), (2048, 2)])
def test_wide_fanouts_one_wave_per_row(mods, fanouts):
    rng = np.random.default_rng(5)
    rowptr, col = random_csr(6000, 60.0, rng)       # skewed: some rows have thousands of entries
    assert np.diff(rowptr).max() > 2048
    batches = random_batches(6000, 3, 70, rng)
    _run_both(mods, rowptr, col, batches, fanouts, 11)


def test_fanout_at_least_max_degree_is_exact(mods):
    rng = np.random.default_rng(6)
    rowptr, col = random_csr(3000, 10.0, rng)
    maxdeg = int(np.diff(rowptr).max())
    batches = random_batches(3000, 4, 33, rng)
    for fan in ((maxdeg, maxdeg), (2**31 - 1, maxdeg + 7)):
        _, res, ref = _run_both(mods, rowptr, col, batches, fan, 1)
        # no randomness: a different seed gives the same result
        _, res2, _ = _run_both(mods, rowptr, col, batches, fan, 2)
        assert torch.equal(res.hop(1).col, res2.hop(1).col)


def test_host_csr_host_batches_directed_with_loops(mods):
    O, bms, _ = mods
    rng = np.random.default_rng(8)
    rowptr, col = random_csr(5000, 9.0, rng, symmetric=False, allow_loops=True)
    batches = random_batches(5000, 6, 40, rng)
    csr = bms.Csr(torch.from_numpy(rowptr), torch.from_numpy(col))           # host arrays, copied
    res = bms.sample_nodewise(csr, batches, (6, 4), 21)                       # host batches
    assert_hops_equal(res.hops(), O.sample_nodewise(rowptr, col, batches, (6, 4), 21))


def test_bulk_equals_stack_and_recycle(mods):
    O, bms, _ = mods
    rng = np.random.default_rng(9)
    rowptr, col = random_csr(8000, 16.0, rng)
    batches = random_batches(8000, 6, 100, rng)
    csr, bulk, ref = _run_both(mods, rowptr, col, batches, (7, 5), 5, mb_base=40)
    res = None
    for i in range(6):        # k = 1 calls with the minibatch index advanced, reusing one result
        res = bms.sample_nodewise(csr, torch.from_numpy(batches[i:i + 1]).cuda(), (7, 5), 5, mb_base=40 + i,
                                  recycle=res)
        one = O.sample_nodewise(rowptr, col, batches[i:i + 1], (7, 5), 5, 40 + i)
        assert_hops_equal(res.hops(), one, what="minibatch %d alone" % i)
        for h in range(2):
            r0, r1 = ref[h].mb_coloff[i], ref[h].mb_coloff[i + 1]
            assert np.array_equal(res.hop(h).col_vertex.cpu().numpy(), ref[h].col_vertex[r0:r1])
    # the same csr handle keeps working for a larger call afterwards (scratch regrown, sets clean)
    res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (7, 5), 5, mb_base=40, recycle=res)
    assert_hops_equal(res.hops(), ref)


def test_degenerate_graphs_and_empty_frontiers(mods):
    O, bms, _ = mods
    # isolated vertices, a hop whose frontier becomes empty, a graph with no edges at all
    rowptr = np.array([0, 0, 1, 1, 1], dtype=np.int64)
    col = np.array([2], dtype=np.int32)
    batches = np.array([[0, 1], [2, 0], [3, 2]], dtype=np.int32)
    _run_both(mods, rowptr, col, batches, (3, 3, 3), 1)
    rowptr0 = np.zeros(11, dtype=np.int64)
    col0 = np.zeros(0, dtype=np.int32)
    _run_both(mods, rowptr0, col0, np.array([[1, 2, 3]], dtype=np.int32), (2, 2), 1)
    # one vertex, one self-loop
    _run_both(mods, np.array([0, 1], dtype=np.int64), np.array([0], dtype=np.int32),
              np.array([[0]], dtype=np.int32), (1, 1), 1)


def test_error_codes(mods):
    O, bms, _ = mods
    rng = np.random.default_rng(10)
    rowptr, col = random_csr(500, 8.0, rng)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    good = random_batches(500, 2, 8, rng)
    for bad, code in ((np.array([[1, 2, 1, 3]], dtype=np.int32), bms.ERANGE),
                      (np.array([[1, 500]], dtype=np.int32), bms.ERANGE),
                      (np.array([[-1, 4]], dtype=np.int32), bms.ERANGE)):
        with pytest.raises(bms.BmsError) as e:
            bms.sample_nodewise(csr, bad, (2,), 1)
        assert e.value.code == code
        # the handle is still usable and the vertex sets are clean again
        res = bms.sample_nodewise(csr, good, (3, 2), 4)
        assert_hops_equal(res.hops(), O.sample_nodewise(rowptr, col, good, (3, 2), 4))
    with pytest.raises(bms.BmsError) as e:
        bms.sample_nodewise(csr, good, (3, 0), 1)
    assert e.value.code == bms.EINVAL
    big = int(np.diff(rowptr).max())
    # malformed matrices are refused at load time
    unsorted = col.copy()
    v = int(np.argmax(np.diff(rowptr)))
    unsorted[rowptr[v]], unsorted[rowptr[v] + 1] = unsorted[rowptr[v] + 1], unsorted[rowptr[v]]
    dup = col.copy()
    dup[rowptr[v] + 1] = dup[rowptr[v]]
    oob = col.copy()
    oob[3] = 500
    badptr = rowptr.copy()
    badptr[5] = badptr[6] + 1
    for rp, cl in ((rowptr, unsorted), (rowptr, dup), (rowptr, oob), (badptr, col)):
        with pytest.raises(bms.BmsError) as e:
            bms.Csr(torch.from_numpy(rp).cuda(), torch.from_numpy(cl).cuda())
        assert e.value.code == bms.EFORMAT, big


def test_profile_stages_are_reported(mods):
    O, bms, _ = mods
    rng = np.random.default_rng(12)
    rowptr, col = random_csr(4000, 12.0, rng)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = bms.sample_nodewise(csr, random_batches(4000, 4, 64, rng), (5, 5), 3, profile=True)
    names = [s[0] for s in res.stages()]
    assert names.count("nw_sample") == 2 and all(s[2] >= 0 for s in res.stages())
    assert len(set(names)) > 3
    # the cheap mode times the sampling kernel only; without a profile flag nothing is recorded
    res = bms.sample_nodewise(csr, random_batches(4000, 4, 64, rng), (5, 5), 3, profile="main", recycle=res)
    assert [(s[0], s[1]) for s in res.stages()] == [("nw_sample", 0), ("nw_sample", 1)]
    assert all(s[2] > 0 for s in res.stages())
    lad = bms.sample_ladies(csr, random_batches(4000, 4, 64, rng), (20,), 3, profile="main")
    assert [s[0] for s in lad.stages()] == ["ldw_accumulate"]
    res = bms.sample_nodewise(csr, random_batches(4000, 4, 64, rng), (5, 5), 3, recycle=res)
    assert res.stages() == []


def test_bucket_extract_many_buckets_and_large_batches(mods):
    # vertex range spanning many 2^18-id buckets, sparse so that most buckets hold a few ids;
    # b above the LDS seed-sort limit exercises the vertex-set seed check next to bucket EXTRACT
    O, bms, _ = mods
    rng = np.random.default_rng(44)
    n = 3_000_000
    src = rng.integers(0, n, size=400_000)
    dst = rng.integers(0, n, size=400_000)
    keep = src != dst
    key = np.unique(np.concatenate([src[keep] * n + dst[keep], dst[keep] * n + src[keep]]))
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.add.at(rowptr, key // n + 1, 1)
    rowptr = np.cumsum(rowptr)
    col = (key % n).astype(np.int32)
    nonisolated = np.nonzero(np.diff(rowptr))[0]
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    for k, b in ((3, 9000), (7, 500)):
        batches = random_batches(n, k, b, rng, candidates=nonisolated)
        ref = O.sample_nodewise(rowptr, col, batches, (3, 3, 2), 5)
        for extract in ("sort", "buckets", "bitmap", None):
            res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (3, 3, 2), 5, extract=extract)
            assert_hops_equal(res.hops(), ref, what="extract=%s k=%d b=%d" % (extract, k, b))
    # repeated seed found by the LDS sort check (b <= 8192) and by the vertex-set check (b > 8192)
    for b in (500, 9000):
        bad = random_batches(n, 2, b, rng)
        bad[1, b - 1] = bad[1, 0]
        with pytest.raises(bms.BmsError) as e:
            bms.sample_nodewise(csr, bad, (2,), 1, extract="buckets")
        assert e.value.code == bms.ERANGE
    bad = random_batches(n, 2, 100, rng)
    bad[0, 7] = n
    with pytest.raises(bms.BmsError) as e:
        bms.sample_nodewise(csr, bad, (2,), 1, extract="buckets")
    assert e.value.code == bms.ERANGE


def test_sort_extract_falls_back_when_ids_crowd_one_segment(mods):
    # directed graph whose edges all point into a narrow id range: every sampled id of a minibatch lands in one
    # id-range segment, more than a segment may hold -> the per-minibatch kernel runs
    O, bms, _ = mods
    rng = np.random.default_rng(45)
    n, m = 1_000_000, 8_000_000
    src = rng.integers(0, n, size=m)
    dst = rng.integers(1030, 2000, size=m)     # narrower than any segment the library would pick
    key = np.unique(src * n + dst)
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.add.at(rowptr, key // n + 1, 1)
    rowptr = np.cumsum(rowptr)
    col = (key % n).astype(np.int32)
    sources = np.nonzero(np.diff(rowptr))[0]
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    batches = random_batches(n, 3, 12000, rng, candidates=sources)
    ref = O.sample_nodewise(rowptr, col, batches, (8, 2), 9)
    per_mb = np.diff(ref[0].rowptr[ref[0].mb_rowoff])
    assert per_mb.min() > 65535       # more pairs in the one segment than a segment may hold
    for extract in ("sort", "buckets", "bitmap"):
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (8, 2), 9, extract=extract)
        assert_hops_equal(res.hops(), ref, what="extract=%s" % extract)


def test_recycled_calls_without_host_round_trips(mods):
    # a recycled result of the same call shape lets the library enqueue all hops without reading sizes
    # back; the second call here samples far more edges than the first (high-degree seeds), a third
    # far fewer, so buffers must be sized by upper bounds and not by the remembered sizes
    O, bms, _ = mods
    rng = np.random.default_rng(46)
    rowptr, col = random_csr(40000, 40.0, rng)
    deg = np.diff(rowptr)
    order = np.argsort(deg)
    low, high = order[:8000], order[-8000:]
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = None
    for pool, seed in ((low, 1), (high, 2), (low, 3), (high, 3)):
        batches = random_batches(40000, 6, 256, rng, candidates=pool)
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (10, 5, 3), seed, recycle=res)
        ref = O.sample_nodewise(rowptr, col, batches, (10, 5, 3), seed)
        assert_hops_equal(res.hops(), ref, what="recycled, seed %d" % seed)
    # an invalid batch on the no-round-trip path is still reported, and the handle recovers
    bad = random_batches(40000, 6, 256, rng)
    bad[2, 5] = bad[2, 6]
    with pytest.raises(bms.BmsError) as e:
        bms.sample_nodewise(csr, torch.from_numpy(bad).cuda(), (10, 5, 3), 4, recycle=res)
    assert e.value.code == bms.ERANGE
    good = random_batches(40000, 6, 256, rng)
    res = bms.sample_nodewise(csr, torch.from_numpy(good).cuda(), (10, 5, 3), 5, recycle=res)
    assert_hops_equal(res.hops(), O.sample_nodewise(rowptr, col, good, (10, 5, 3), 5))


def test_sort_extract_segments_sorted_by_whole_workgroups(mods):
    # most edges point into a few id-range segments, each of which then holds more pairs than one wave
    # sorts (but few enough for one workgroup); the rest spread over the whole id range, so that waves
    # and workgroups both feed the slot lists of the same minibatch
    O, bms, _ = mods
    rng = np.random.default_rng(47)
    n, m = 3_000_000, 900_000
    src = rng.integers(0, n, size=m)
    dst = np.where(rng.random(m) < 0.7, rng.integers(1 << 16, 4 << 16, size=m), rng.integers(0, n, size=m))
    key = np.unique(src * n + dst)
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.add.at(rowptr, key // n + 1, 1)
    rowptr = np.cumsum(rowptr)
    col = (key % n).astype(np.int32)
    sources = np.nonzero(np.diff(rowptr))[0]
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    batches = random_batches(n, 5, 8000, rng, candidates=sources)
    ref = O.sample_nodewise(rowptr, col, batches, (3, 2), 11)
    # sampled ids of minibatch 0 per range of 2^16 ids (the segment width the library picks for this shape)
    e1 = ref[0].rowptr[ref[0].mb_rowoff[1]]
    per_segment = np.bincount(ref[0].col_vertex[ref[0].col[:e1]] >> 16)
    assert 1024 < per_segment.max() <= 4096, per_segment.max()
    for extract in ("sort", None):
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (3, 2), 11, extract=extract)
        assert_hops_equal(res.hops(), ref, what="extract=%s" % extract)


def test_sort_extract_largest_workgroup_sorted_segments(mods):
    # as above with most edges into ONE id range of 2^16: its segment holds several thousand pairs (several tiles
    # of the back-split per segment), ranked by a workgroup through a bitmap in LDS
    O, bms, _ = mods
    rng = np.random.default_rng(49)
    n, m = 3_000_000, 1_200_000
    src = rng.integers(0, n, size=m)
    dst = np.where(rng.random(m) < 0.7, rng.integers(1 << 16, 2 << 16, size=m), rng.integers(0, n, size=m))
    key = np.unique(src * n + dst)
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.add.at(rowptr, key // n + 1, 1)
    rowptr = np.cumsum(rowptr)
    col = (key % n).astype(np.int32)
    sources = np.nonzero(np.diff(rowptr))[0]
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    batches = random_batches(n, 5, 8000, rng, candidates=sources)
    ref = O.sample_nodewise(rowptr, col, batches, (3, 2), 12)
    for i in range(5):
        e0, e1 = ref[0].rowptr[ref[0].mb_rowoff[i]], ref[0].rowptr[ref[0].mb_rowoff[i + 1]]
        per_segment = np.bincount(ref[0].col_vertex[ref[0].mb_coloff[i] + ref[0].col[e0:e1]] >> 16)
        assert 4096 < per_segment.max() <= 16384, per_segment.max()
    for extract in ("sort", None):
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (3, 2), 12, extract=extract)
        assert_hops_equal(res.hops(), ref, what="extract=%s" % extract)


def test_vertex_ids_sorted_by_degree(mods):
    # hubs first: the sampled ids of every minibatch crowd the low end of the id range, so many id-range
    # segments hold far more pairs than a wave sorts and are ranked through LDS bitmaps, others stay small
    O, bms, _ = mods
    rng = np.random.default_rng(50)
    n = 400_000
    rowptr, col = skewed_csr(n, 6_000_000, rng)
    deg = np.diff(rowptr)
    order = np.argsort(-deg, kind="stable")
    newid = np.empty(n, dtype=np.int64)
    newid[order] = np.arange(n)
    src = np.repeat(np.arange(n), deg)
    key = np.sort(newid[src] * n + newid[col])
    rowptr2 = np.zeros(n + 1, dtype=np.int64)
    np.add.at(rowptr2, key // n + 1, 1)
    rowptr2 = np.cumsum(rowptr2)
    col2 = (key % n).astype(np.int32)
    batches = random_batches(n, 6, 2000, rng, candidates=np.nonzero(np.diff(rowptr2) > 0)[0])
    ref = O.sample_nodewise(rowptr2, col2, batches, (10, 5, 3), 13)
    e1 = ref[2].rowptr[ref[2].mb_rowoff[1]]
    first = ref[2].col_vertex[ref[2].col[:e1]]                  # global ids sampled by minibatch 0 at the last hop
    assert (first < n // 100).mean() > 0.08                      # ten times denser among the top 1 % of the ids
    assert np.bincount(first >> 9).max() > 2048                  # far more than a wave sorts, in ranges of 512 ids
    csr = bms.Csr(torch.from_numpy(rowptr2).cuda(), torch.from_numpy(col2).cuda())
    res = None
    for extract in ("sort", None, "buckets"):
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (10, 5, 3), 13, extract=extract, recycle=res)
        assert_hops_equal(res.hops(), ref, what="degree-sorted ids, extract=%s" % extract)


def test_minibatch_with_more_sampled_edges_than_the_slot_lists_cover(mods):
    # one minibatch whose last hop samples more than 256 * 8192 edges: its local columns are stored
    # directly instead of through the per-range slot lists
    O, bms, synth = mods
    g = synth.rmat_graph(1 << 21, 24_000_000, 0.45, 0.22, 0.22, seed=5, device="cuda")
    rowptr, col = g.rowptr.cpu().numpy(), g.col.cpu().numpy()
    rng = np.random.default_rng(48)
    deg = np.diff(rowptr)
    batches = random_batches(g.n, 2, 8000, rng, candidates=np.nonzero(deg >= 8)[0])
    csr = bms.Csr(g.rowptr, g.col)
    ref = O.sample_nodewise(rowptr, col, batches, (15, 10, 5), 3)
    per_mb = np.diff(ref[2].rowptr[ref[2].mb_rowoff])
    assert per_mb.max() > 256 * 8192, per_mb
    res = None
    for extract in ("sort", "buckets", "sort"):
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (15, 10, 5), 3, extract=extract, recycle=res)
        assert_hops_equal(res.hops(), ref, what="extract=%s" % extract)


def test_thousands_of_small_minibatches_and_the_limit_on_k(mods):
    O, bms, _ = mods
    rng = np.random.default_rng(49)
    rowptr, col = random_csr(60000, 9.0, rng)
    batches = random_batches(60000, 3000, 4, rng)
    csr, res, ref = _run_both(mods, rowptr, col, batches, (4, 3), 8)
    lad = bms.sample_ladies(csr, torch.from_numpy(batches).cuda(), (6, 6), 8)
    assert_hops_equal(lad.hops(), O.sample_ladies(rowptr, col, batches, (6, 6), 8), with_p=True)
    with pytest.raises(bms.BmsError) as e:
        bms.sample_nodewise(csr, torch.zeros((65536, 1), dtype=torch.int32).cuda(), (2,), 1)
    assert e.value.code == bms.EINVAL


def test_side_stream_and_graph_without_vertices(mods):
    O, bms, _ = mods
    rng = np.random.default_rng(50)
    rowptr, col = random_csr(20000, 10.0, rng)
    batches = random_batches(20000, 6, 100, rng)
    ref = O.sample_nodewise(rowptr, col, batches, (6, 4), 2)
    lref = O.sample_ladies(rowptr, col, batches, (50, 50), 2)
    side = torch.cuda.Stream()  # default priority
    with torch.cuda.stream(side):
        csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
        dev = torch.from_numpy(batches).cuda()
        res = None
        for _ in range(3):
            res = bms.sample_nodewise(csr, dev, (6, 4), 2, recycle=res)
        lad = bms.sample_ladies(csr, dev, (50, 50), 2)
        X = bms.fetch_features(torch.ones((20000, 8), device="cuda"), res.hop(1).col_vertex)
        Y = bms.aggregate_hop(res, 1, X)
    side.synchronize()
    assert_hops_equal(res.hops(), ref, what="side stream")
    assert_hops_equal(lad.hops(), lref, with_p=True, what="side stream")
    assert torch.equal(Y.cpu(), (torch.from_numpy(np.diff(ref[1].rowptr)) > 0).float()[:, None].repeat(1, 8))
    # a matrix with no vertices loads; every seed is then out of range
    empty = bms.Csr(torch.zeros(1, dtype=torch.int64).cuda(), torch.zeros(0, dtype=torch.int32).cuda())
    for fn in (bms.sample_nodewise, bms.sample_ladies):
        with pytest.raises(bms.BmsError) as e:
            fn(empty, np.zeros((1, 1), dtype=np.int32), (2,), 1)
        assert e.value.code == bms.ERANGE


def _hub_graph(n, hub_share, rng):
    """Directed graph: every vertex points at one random vertex, and a share of them also at one hub."""
    hub = 12345
    dst = rng.integers(0, n, size=n)
    dst[dst == np.arange(n)] = (dst[dst == np.arange(n)] + 1) % n
    has_hub = rng.random(n) < hub_share
    has_hub[hub] = False
    has_hub &= dst != hub
    deg = 1 + has_hub.astype(np.int64)
    rowptr = np.zeros(n + 1, dtype=np.int64)
    rowptr[1:] = np.cumsum(deg)
    col = np.empty(rowptr[-1], dtype=np.int32)
    first = np.where(has_hub, np.minimum(dst, hub), dst)
    col[rowptr[:-1]] = first
    col[rowptr[:-1][has_hub] + 1] = np.maximum(dst, hub)[has_hub]
    return rowptr, col, hub


@pytest.mark.parametrize("b,hub_share,what", [
    (16000, 0.02, "one id in more than 32 rows of a segment that one workgroup ranks: handed to the bitmap kernel"),
    (16000, 0.6, "the hub's segment holds more ids than one workgroup ranks: listed for the bitmap kernel"),
    (900, 0.2, "segments wider than the bitmap kernel takes: the per-minibatch kernel redoes the hop"),
])
def test_sort_extract_one_vertex_sampled_by_many_rows(mods, b, hub_share, what):
    # sparse hop (far fewer sampled ids than vertices): the ids of a segment are ranked by counting them into buckets
    # of about one id; a hub that many rows of a minibatch sample crowds one bucket
    O, bms, _ = mods
    rng = np.random.default_rng(51)
    n = 1 << 22
    rowptr, col, hub = _hub_graph(n, hub_share, rng)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    batches = random_batches(n, 3, b, rng)
    ref = O.sample_nodewise(rowptr, col, batches, (2, 1), 21)
    picked = ref[0].col_vertex[ref[0].col[:ref[0].rowptr[ref[0].mb_rowoff[1]]]]
    assert (picked == hub).sum() > 32, what
    for extract in ("sort", None, "buckets"):
        res = None
        for _ in range(2):   # the second call runs without host round trips
            res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (2, 1), 21, extract=extract, recycle=res)
            assert_hops_equal(res.hops(), ref, what="%s, extract=%s" % (what, extract))


def test_sort_extract_dense_hops_ranked_by_bitmap_with_many_duplicates(mods):
    # dense hop (a minibatch samples a large share of the vertices): every segment is ranked through a bitmap of
    # its id range; most ids are sampled several times, segments hold tens of thousands of ids
    O, bms, _ = mods
    rng = np.random.default_rng(52)
    n = 60000
    rowptr, col = random_csr(n, 30.0, rng)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    batches = random_batches(n, 4, 6000, rng)
    ref = O.sample_nodewise(rowptr, col, batches, (8, 4), 22)
    assert ref[1].nnz / 4 > 50000 and ref[1].nnz > 2 * ref[1].ncols
    for extract in ("sort", None):
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (8, 4), 22, extract=extract)
        assert_hops_equal(res.hops(), ref, what="extract=%s" % extract)


@pytest.mark.parametrize("b", [1023, 1024, 1025, 2048, 3072])
def test_sort_extract_minibatches_that_fill_tiles_of_the_cut_exactly(mods, b):
    # every vertex has 10 neighbours, fanout 8: a minibatch samples exactly 8 b ids, i.e. one short of, exactly, or
    # one more than whole tiles of 8192 positions of the cut; the second hop (fanout 2) does the same on distinct ids
    O, bms, _ = mods
    n = 150_000
    v = np.arange(n, dtype=np.int64)
    nb = np.stack([(v + d) % n for d in (-5, -4, -3, -2, -1, 1, 2, 3, 4, 5)], axis=1)
    nb.sort(axis=1)
    rowptr = np.arange(n + 1, dtype=np.int64) * 10
    col = nb.reshape(-1).astype(np.int32)
    rng = np.random.default_rng(b)
    batches = random_batches(n, 3, b, rng)
    ref = O.sample_nodewise(rowptr, col, batches, (8, 2), 31)
    assert ref[0].nnz == 3 * 8 * b
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = None
    for _ in range(2):
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (8, 2), 31, extract="sort", recycle=res)
        assert_hops_equal(res.hops(), ref, what="b=%d" % b)


@pytest.mark.parametrize("n,k,b,fanouts,stages", [
    (4000, 4, 64, (5, 5), ["nw_small"]),                                          # every hop in one launch
    (4000, 40, 500, (20, 10), ["nw_small", "nw_rows", "scan_tiles", "nw_sample", "rg_mark", "rg_emit", "rg_lookup"]),
    (200_000, 2, 900, (15, 10), ["nw_small", "nw_rows", "scan_tiles", "nw_sample", "rg_count", "rg_emit_gather"])])
def test_calls_timed_as_they_run(mods, n, k, b, fanouts, stages):
    # the stages are those of the kernels that a call without a profile runs
    O, bms, _ = mods
    rng = np.random.default_rng(n + k)
    rowptr, col = random_csr(n, 14.0, rng)
    batches = random_batches(n, k, b, rng)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    ref = O.sample_nodewise(rowptr, col, batches, fanouts, 3)
    res = None
    for profile in ("as_run", "as_run", "main_as_run", False):
        res = bms.sample_nodewise(csr, batches, fanouts, 3, profile=profile, recycle=res)
        names = [s[0] for s in res.stages()]
        if profile == "as_run":
            assert [x for x in names if x != "seeds"] == stages and all(s[2] >= 0 for s in res.stages())
        else:
            assert names == (["nw_sample"] if profile and "nw_sample" in stages else [])
        assert_hops_equal(res.hops(), ref, what="n=%d k=%d profile=%s" % (n, k, profile))


def test_result_recycled_with_another_graph_at_the_address_of_the_old_one(mods):
    # what a result remembers (sizes, kernel paths, the table of unequal segments) belongs to the handle, not to its address, which
    # the next handle gets after bms_free
    O, bms, _ = mods
    rng = np.random.default_rng(52)

    def hubs_first(n, m):
        rowptr, col = skewed_csr(n, m, rng)
        deg = np.diff(rowptr)
        order = np.argsort(-deg, kind="stable")
        newid = np.empty(n, dtype=np.int64)
        newid[order] = np.arange(n)
        key = np.sort(newid[np.repeat(np.arange(n), deg)] * n + newid[col])
        rowptr = np.zeros(n + 1, dtype=np.int64)
        np.add.at(rowptr, key // n + 1, 1)
        return np.cumsum(rowptr), (key % n).astype(np.int32)

    graphs = []
    for n, m in ((6_000_000, 5_000_000), (9_000_000, 7_000_000), (5_500_000, 5_000_000)):
        rowptr, col = hubs_first(n, m)
        batches = random_batches(n, 3, 2000, rng, candidates=np.nonzero(np.diff(rowptr) > 0)[0])
        graphs.append((torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda(), batches,
                       O.sample_nodewise(rowptr, col, batches, (10, 8, 6), 13)))
    res, address = None, None
    for g, (rowptr, col, batches, ref) in enumerate(graphs):
        handles = [bms.Csr(rowptr, col) for _ in range(20)]
        pick = [c for c in handles if c.handle.value == address] or handles[:1]
        address = pick[0].handle.value
        for call in range(3):
            res = bms.sample_nodewise(pick[0], batches, (10, 8, 6), 13, extract="sort", recycle=res)
            assert (res.attempts() > 1) == (call == 0), "graph %d, call %d: %d attempts" % (g, call, res.attempts())
            assert_hops_equal(res.hops(), ref, what="graph %d call %d" % (g, call))
        for c in handles:
            c.free()


@pytest.mark.parametrize("k,replace", [(1, False), (7, False), (7, True), (40, False)])
def test_row_tiles_of_minibatches_of_very_different_size(mods, k, replace):
    # second-hop frontiers of no row, one tile and dozens side by side: every tile is visited once, whatever the share of steps
    # that its minibatch has
    O, bms, _ = mods
    rng = np.random.default_rng(k)
    n, b = 60_000, 500
    degree = np.zeros(n, dtype=np.int64)
    for i in range(k): # seeds of minibatch i: ids from i b on
        degree[i * b:(i + 1) * b] = [0, 1, 3, 40, 40, 0, 12][(i + 3) % 7]
    degree[k * b:] = rng.integers(0, 6, n - k * b)
    rowptr = np.concatenate([[0], np.cumsum(degree)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(n, d, replace=False)) for d in degree]).astype(np.int32)
    batches = np.arange(k * b, dtype=np.int32).reshape(k, b)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    ref = O.sample_nodewise(rowptr, col, batches, (30, 4, 3), 5, replace=replace)
    for extract in ("sort", "bitmap"):
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (30, 4, 3), 5, extract=extract, replace=replace)
        assert_hops_equal(res.hops(), ref, what="extract=%s" % extract)


@pytest.mark.parametrize("hub", [False, True])
@pytest.mark.parametrize("b,fanouts,union_dst", [(1024, (1, 1, 1), False), (205, (5, 3), False), (93, (10, 15), True), (1024, (4, 4), False),
                                                 (1025, (4, 3), True), (1024, (16,), False), (963, (16,), True), (5, (7, 9, 11), False)])
def test_one_workgroup_hops_around_their_round_counts(mods, b, fanouts, union_dst, hub):
    # a thread keeps 1, up to 4 or up to 16 entries of 1024 each; `hub`: a vertex that every row has, which crowds its bucket, so
    # that the hop is ranked by the sort, in between hops that are not
    O, bms, _ = mods
    rng = np.random.default_rng(b)
    n, degree = 40_000, 16
    rows = [rng.choice(n // 2 - 20, degree, replace=False) + 20 for _ in range(n)]
    if hub:
        for r in rows[:n // 2]: # (17 is in no row otherwise)
            r[rng.integers(degree)] = 17
    rowptr = np.arange(n + 1, dtype=np.int64) * degree
    col = np.concatenate([np.sort(r) for r in rows]).astype(np.int32)
    batches = np.stack([rng.permutation(n)[:b] for _ in range(3)]).astype(np.int32)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    for replace in (False, True):
        ref = O.sample_nodewise(rowptr, col, batches, fanouts, 3, 1, union_dst=union_dst, replace=replace)
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), fanouts, 3, mb_base=1, union_dst=union_dst, replace=replace)
        assert_hops_equal(res.hops(), ref, what="replace=%s" % replace)


@pytest.mark.parametrize("s", [33, 48, 49, 64])
@pytest.mark.parametrize("k,variant", [(2, {}), (9, {}), (9, dict(union_dst=True))])
def test_wide_fanouts_one_lane_per_row(mods, s, k, variant):
    # so many rows (65536 by their bound) that fanouts of 33 .. 64 are drawn one row per lane; degrees around s, ragged tiles;
    # k = 2: the sampling kernel sets bits
    O, bms, _ = mods
    rng = np.random.default_rng(s)
    n, b = 40_000, 8192 // k + 5
    degree = rng.choice([0, 1, s - 1, s, s + 1, 90], n)
    rowptr = np.concatenate([[0], np.cumsum(degree)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(n, d, replace=False)) for d in degree]).astype(np.int32)
    batches = random_batches(n, k, b, rng)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    ref = O.sample_nodewise(rowptr, col, batches, (8, s), 11, **variant)
    for extract in (None, "sort", "bitmap"):
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (8, s), 11, extract=extract, **variant)
        assert_hops_equal(res.hops(), ref, what="extract=%s" % extract)


@pytest.mark.parametrize("n", [2047, 2048, 2049, 6145, 131_200])
@pytest.mark.parametrize("k", [1, 5, 40])
def test_vertex_ranges_written_out_wave_by_wave(mods, n, k):
    # columns leave in steps of 2048 ids: nearly all vertices sampled (small n, up to all ids of a step), few of them (large n)
    rng = np.random.default_rng(n + k)
    degree = 40
    col = np.concatenate([np.sort(rng.choice(n, degree, replace=False)) for _ in range(n)]).astype(np.int32)
    rowptr = np.arange(n + 1, dtype=np.int64) * degree
    batches = random_batches(n, k, 1100, rng)
    O, bms, _ = mods
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (16, 20), 2)
    assert_hops_equal(res.hops(), O.sample_nodewise(rowptr, col, batches, (16, 20), 2))


@pytest.mark.parametrize("share,spread", [(1.0, 1), (0.5, 3), (0.2, 700)])
def test_sort_extract_buckets_of_equal_and_near_ids(mods, share, spread):
    # buckets of 1 to 32 ids, many of them equal or next to each other, at the ends of segments and of the id range
    O, bms, _ = mods
    rng = np.random.default_rng(spread)
    n, b = 900_000, 900
    near = (rng.integers(0, n // 1000, 400) * 1000 + rng.integers(0, spread, 400)) % n
    near[:4] = (0, 1, n - 2, n - 1)
    rows = []
    for _ in range(b):
        r = rng.choice(n, 24, replace=False)
        m = int(24 * share * 0.5)
        r[:m] = rng.choice(near, m)
        rows.append(np.unique(r))
    deg = np.zeros(n, dtype=np.int64)
    deg[:b] = [r.size for r in rows]
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    col = np.concatenate(rows).astype(np.int32)
    batches = np.stack([rng.permutation(b) for _ in range(5)]).astype(np.int32)
    _run_both(mods, rowptr, col, batches, (20,), 3)


@pytest.mark.parametrize("k,b,fanouts", [(1, 300, (16, 16, 2)), (1, 1, (17, 40)), (5, 2000, (17, 3)), (4, 16000, (17, 2)), (5, 600, (40, 33))])
def test_tiles_summed_by_the_sampling_kernel(mods, k, b, fanouts):
    # recycled calls: 1 to 1024 tiles of rows and more, one row per lane and per wave; no rows at all (seeds without neighbours)
    rng = np.random.default_rng(b)
    n = 70_000
    degree = rng.integers(0, 60, n)
    degree[:3000] = 0
    rowptr = np.concatenate([[0], np.cumsum(degree)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(n, d, replace=False)) for d in degree]).astype(np.int32)
    O, bms, _ = mods
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = None
    for seed, pool in ((1, np.arange(n)), (2, np.arange(n)), (3, np.arange(3000) if k * b <= 3000 else np.arange(n)), (4, np.arange(n))):
        batches = random_batches(n, k, b, rng, candidates=pool)
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), fanouts, seed, recycle=res)
        assert_hops_equal(res.hops(), O.sample_nodewise(rowptr, col, batches, fanouts, seed), what="seed=%d" % seed)


@pytest.mark.parametrize("k,n", [(1025, 3000), (400, 400_000), (100, 1_400_000)])
def test_column_offsets_of_many_minibatches_and_ranges(mods, k, n):
    # around 1024 pairs of (minibatch, range of ids), which are placed at once up to there
    rng = np.random.default_rng(k)
    degree = 30
    rows = rng.permutation(n)[:2000]
    deg = np.zeros(n, dtype=np.int64)
    deg[rows] = degree
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(n, degree, replace=False)) for _ in range(2000)]).astype(np.int32)
    batches = random_batches(n, k, 20 if k > 1024 else 700, rng, candidates=rows)
    O, bms, _ = mods
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (25, 4), 6)
    assert_hops_equal(res.hops(), O.sample_nodewise(rowptr, col, batches, (25, 4), 6))


@pytest.mark.parametrize("n,k,b,fanouts", [(1_300_000, 6, 200, (40,)), (4_900_000, 5, 150, (33, 2)), (2_000_000, 74, 104, (40,)), (2_000_000, 76, 104, (40,))])
@pytest.mark.parametrize("variant", [{}, dict(union_dst=True), dict(replace=True)], ids=lambda v: "+".join(v))
def test_hops_whose_bitmaps_are_small_go_by_ranges(mods, n, k, b, fanouts, variant):
    # many more than 64 ids of [0, n) per entry: by ranges up to 150 million ids in all minibatches' bitmaps (and the same
    # just above), entries at both ends of the id range
    rng = np.random.default_rng(n + k)
    rows = np.unique(np.concatenate([[0, n - 1], rng.choice(n, 1500, replace=False)]))
    deg = np.zeros(n, dtype=np.int64)
    deg[rows] = rng.integers(30, 60, rows.size)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    parts = []
    for d in deg[rows]:
        c = np.unique(np.concatenate([rng.choice(n, d - 2, replace=False), [0, n - 1]]))
        while c.size < d:
            c = np.unique(np.append(c, rng.integers(0, n)))
        parts.append(c)
    col = np.concatenate(parts).astype(np.int32)
    batches = random_batches(n, k, b, rng, candidates=rows)
    O, bms, _ = mods
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    ref = O.sample_nodewise(rowptr, col, batches, fanouts, 8, **variant)
    res = None
    for _ in range(2):
        res = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), fanouts, 8, recycle=res, **variant)
        assert_hops_equal(res.hops(), ref)
