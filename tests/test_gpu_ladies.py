"""Parity of the HIP layer-wise (LADIES) sampler with the CPU oracle (bit-exact), through the C ABI."""
import numpy as np
import pytest
import torch

from conftest import random_batches, random_csr
from parity import assert_hops_equal

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mods():
    from oracle import bms_oracle as O
    from paper_2311_02909_amd import bms, synth
    assert torch.cuda.is_available()
    return O, bms, synth


def _run_both(mods, rowptr, col, batches, s_per_layer, seed, mb_base=0, squared=False, csr=None):
    O, bms, _ = mods
    if csr is None:
        csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    ref = O.sample_ladies(rowptr, col, batches, s_per_layer, seed, mb_base, squared)
    # the kernel paths: counters in HBM; counters in LDS windows, the rows' window boundaries found per hop;
    # the same with the boundaries copied from the per-graph index (built by the first call that may use it)
    for dense, index in ((True, True), (False, False), (False, True)):
        res = bms.sample_ladies(csr, torch.from_numpy(batches).cuda(), s_per_layer, seed, mb_base=mb_base,
                                squared=squared, dense=dense, index=index)
        assert_hops_equal(res.hops(), ref, with_p=True,
                          what="s=%s seed=%d squared=%s dense=%s index=%s" % (s_per_layer, seed, squared, dense, index))
    return csr, res, ref


def test_tiny_graph_layerwise(mods):
    O, bms, synth = mods
    g, batches, _ = synth.make_workload("tiny_sage")
    _run_both(mods, g.rowptr.numpy(), g.col.numpy(), batches.numpy(), (64, 64), synth.SAMPLING_SEED)


@pytest.mark.parametrize("s,squared", [((1,), False), ((16, 16), False), ((100, 50, 25), False), ((512, 512, 512), False),
                                       ((64, 64), True), ((3000, 10), True), ((4096, 4097, 5), False)])
def test_random_graph(mods, s, squared):
    # gathered order spans many 4096-entry tiles with a ragged tail; P spans several chunks and tiles
    rng = np.random.default_rng(len(s) * 100 + s[0])
    rowptr, col = random_csr(30000, 30.0, rng)
    batches = random_batches(30000, 5, 200, rng)
    _run_both(mods, rowptr, col, batches, s, 17, mb_base=2, squared=squared)


@pytest.mark.parametrize("s,squared", [((400, 300, 200), False), ((2000, 50), True)])
def test_many_id_windows(mods, s, squared):
    # vertex ids span several 2^16-id windows; a skewed graph, so hub rows cross every window and
    # leaf rows cross none
    O, bms, synth = mods
    g = synth.rmat_graph(300_000, 2_000_000, 0.55, 0.2, 0.2, seed=9, device="cuda")
    rowptr, col = g.rowptr.cpu().numpy(), g.col.cpu().numpy()
    rng = np.random.default_rng(s[0])
    batches = random_batches(g.n, 6, 300, rng)
    _run_both(mods, rowptr, col, batches, s, 23, mb_base=1, squared=squared, csr=bms.Csr(g.rowptr, g.col))


def test_directed_with_loops_and_host_inputs(mods):
    O, bms, _ = mods
    rng = np.random.default_rng(31)
    rowptr, col = random_csr(5000, 9.0, rng, symmetric=False, allow_loops=True)
    batches = random_batches(5000, 6, 40, rng)
    csr = bms.Csr(torch.from_numpy(rowptr), torch.from_numpy(col))
    res = bms.sample_ladies(csr, batches, (30, 30), 21)
    assert_hops_equal(res.hops(), O.sample_ladies(rowptr, col, batches, (30, 30), 21), with_p=True)


def test_bulk_equals_stack_recycle_and_mixed_calls(mods):
    O, bms, _ = mods
    rng = np.random.default_rng(32)
    rowptr, col = random_csr(8000, 16.0, rng)
    batches = random_batches(8000, 4, 64, rng)
    csr, bulk, ref = _run_both(mods, rowptr, col, batches, (40, 40), 5, mb_base=9)
    res = None
    for i in range(4):
        res = bms.sample_ladies(csr, torch.from_numpy(batches[i:i + 1]).cuda(), (40, 40), 5, mb_base=9 + i, recycle=res)
        assert_hops_equal(res.hops(), O.sample_ladies(rowptr, col, batches[i:i + 1], (40, 40), 5, 9 + i), with_p=True)
    # node-wise and layer-wise calls share the handle's vertex sets: interleave them
    nw = bms.sample_nodewise(csr, torch.from_numpy(batches).cuda(), (5, 5), 3)
    assert_hops_equal(nw.hops(), O.sample_nodewise(rowptr, col, batches, (5, 5), 3))
    _run_both(mods, rowptr, col, batches, (40, 40), 6, csr=csr)


def test_degenerate_inputs_and_errors(mods):
    O, bms, _ = mods
    rowptr = np.array([0, 0, 0, 1, 2], dtype=np.int64)
    col = np.array([3, 2], dtype=np.int32)
    _run_both(mods, rowptr, col, np.array([[0, 1], [2, 0]], dtype=np.int32), (2, 2, 2), 1)
    _run_both(mods, np.zeros(6, dtype=np.int64), np.zeros(0, dtype=np.int32), np.array([[1, 2]], dtype=np.int32),
              (3, 3), 1)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    for bad in (np.array([[1, 1]], dtype=np.int32), np.array([[0, 4]], dtype=np.int32)):
        with pytest.raises(bms.BmsError) as e:
            bms.sample_ladies(csr, bad, (2,), 1)
        assert e.value.code == bms.ERANGE
    _run_both(mods, rowptr, col, np.array([[3, 2]], dtype=np.int32), (1,), 1, csr=csr)
    with pytest.raises(bms.BmsError) as e:
        bms.sample_ladies(csr, np.array([[3, 2]], dtype=np.int32), (1,), 1, scratch_limit=8)
    assert e.value.code == bms.ENOMEM


def test_paper_worked_example_on_the_gpu(mods):
    # Sec. 2.2: batch {1,5}; e = [1,0,1,1,2,0]; with squared weights the array is [1,0,1,1,4,0]/7
    O, bms, _ = mods
    edges = [(0, 1), (2, 1), (3, 5), (4, 1), (4, 5)]
    A = np.zeros((6, 6), dtype=np.int64)
    for u, v in edges:
        A[u, v] = A[v, u] = 1
    rowptr = np.concatenate([[0], np.cumsum(A.sum(axis=1))]).astype(np.int64)
    col = np.concatenate([np.nonzero(A[v])[0] for v in range(6)]).astype(np.int32)
    batch = np.array([[1, 5]], dtype=np.int32)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    for seed in range(20):
        res = bms.sample_ladies(csr, batch, (2,), seed, squared=True)
        hop = res.hop(0).to_host()
        e = np.zeros(6, dtype=np.int64)
        e[hop.p_col] = hop.p_cnt
        assert e.tolist() == [1, 0, 1, 1, 2, 0]
        assert_hops_equal([hop], O.sample_ladies(rowptr, col, batch, (2,), seed, squared=True), with_p=True)


@pytest.mark.parametrize("b", [8192, 9000])
def test_largest_batches_of_each_kernel_path(mods, b):
    # b = 8192 is the most the LDS-window path takes (seed check by an LDS sort, 16-bit counters); larger batches
    # run on the dense-counter path by themselves
    O, bms, synth = mods
    g = synth.rmat_graph(120_000, 700_000, 0.5, 0.2, 0.2, seed=11, device="cuda")
    rowptr, col = g.rowptr.cpu().numpy(), g.col.cpu().numpy()
    rng = np.random.default_rng(b)
    batches = random_batches(g.n, 2, b, rng)
    ref = O.sample_ladies(rowptr, col, batches, (300, 100), 4)
    res = bms.sample_ladies(bms.Csr(g.rowptr, g.col), torch.from_numpy(batches).cuda(), (300, 100), 4)
    assert_hops_equal(res.hops(), ref, with_p=True, what="b=%d" % b)


def test_window_index_is_built_once_when_it_fits_and_left_out_when_it_does_not(mods):
    # the index of where adjacency lists cross the window boundaries: n * (windows + 1) 32-bit words held by the
    # handle after the first call that may build it; not built under BMS_LADIES_NO_INDEX, with a scratch limit
    # whose quarter it exceeds, or for a graph whose column array is less than half its size; same results always
    O, bms, synth = mods
    g = synth.rmat_graph(300_000, 2_000_000, 0.55, 0.2, 0.2, seed=5, device="cuda")
    rowptr, col = g.rowptr.cpu().numpy(), g.col.cpu().numpy()
    rng = np.random.default_rng(77)
    batches = random_batches(g.n, 4, 200, rng)
    s = (150, 100)
    ref = O.sample_ladies(rowptr, col, batches, s, 8)
    index_bytes = g.n * ((g.n + 65535) // 65536 + 1) * 4
    dev_batches = torch.from_numpy(batches).cuda()

    csr = bms.Csr(g.rowptr, g.col)
    res = bms.sample_ladies(csr, dev_batches, s, 8, index=False)
    assert_hops_equal(res.hops(), ref, with_p=True, what="no index")
    without = csr.held_bytes()
    res = bms.sample_ladies(csr, dev_batches, s, 8)
    assert_hops_equal(res.hops(), ref, with_p=True, what="index built by this call")
    held = csr.held_bytes()
    assert held >= without + index_bytes - (g.n * 6 * 4) // 2  # the per-hop lists shrink to half without their row-major copy
    res = bms.sample_ladies(csr, dev_batches, s, 8, recycle=res)
    assert_hops_equal(res.hops(), ref, with_p=True, what="index reused")
    assert held <= csr.held_bytes() < held + index_bytes  # (scratch sized with a margin by the recycled call, no second index)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        res = bms.sample_ladies(csr, dev_batches, s, 9, stream=stream.cuda_stream)
    assert_hops_equal(res.hops(), O.sample_ladies(rowptr, col, batches, s, 9), with_p=True, what="index on another stream")

    small = bms.Csr(g.rowptr, g.col)
    res = bms.sample_ladies(small, dev_batches, s, 8, scratch_limit=3 * index_bytes)
    assert_hops_equal(res.hops(), ref, with_p=True, what="scratch limit of three times the index")
    assert small.held_bytes() < index_bytes + without

    # average degree 0.5: the index would be four times the column array
    rng = np.random.default_rng(78)
    rp, cl = random_csr(70_000, 0.5, rng)
    bt = random_batches(70_000, 3, 100, rng)
    sparse = bms.Csr(torch.from_numpy(rp).cuda(), torch.from_numpy(cl).cuda())
    res = bms.sample_ladies(sparse, torch.from_numpy(bt).cuda(), (50, 50), 3)
    assert_hops_equal(res.hops(), O.sample_ladies(rp, cl, bt, (50, 50), 3), with_p=True, what="sparse graph")
    plain = bms.Csr(torch.from_numpy(rp).cuda(), torch.from_numpy(cl).cuda())
    bms.sample_ladies(plain, torch.from_numpy(bt).cuda(), (50, 50), 3, index=False)
    assert sparse.held_bytes() == plain.held_bytes()


def test_recycled_calls_without_size_read_backs_and_their_fallback(mods):
    # a recycled result remembers what its call shape needed (gathered neighbours, nnz(P), kept neighbours per hop):
    # the next call of that shape sizes its buffers from it and checks on the device; when the new seeds need more
    # (hubs instead of leaves) the device flag goes up and the call is repeated with read-backs.  Same results.
    O, bms, synth = mods
    g = synth.rmat_graph(200_000, 3_000_000, 0.57, 0.19, 0.19, seed=21, device="cuda")
    rowptr, col = g.rowptr.cpu().numpy(), g.col.cpu().numpy()
    deg = np.diff(rowptr)
    order = np.argsort(deg, kind="stable")
    k, b, s = 4, 128, (96, 64)
    leaves = order[deg[order] > 0][:k * b].astype(np.int32).reshape(k, b)
    hubs = order[-k * b:].astype(np.int32).reshape(k, b)
    rng = np.random.default_rng(5)
    mixed = random_batches(g.n, k, b, rng)
    csr = bms.Csr(g.rowptr, g.col)
    res = None
    attempts = []
    for step, (batches, seed) in enumerate([(leaves, 1), (leaves, 2), (mixed, 3), (hubs, 4), (hubs, 5), (leaves, 6)]):
        res = bms.sample_ladies(csr, torch.from_numpy(batches).cuda(), s, seed, recycle=res)
        attempts.append(res.attempts())
        assert_hops_equal(res.hops(), O.sample_ladies(rowptr, col, batches, s, seed), with_p=True, what="step %d" % step)
    # leaves gather a few hundred neighbours at the first hop, hubs far more than the margin over that allows: that
    # call repeats itself; the same seeds again then fit what is remembered
    assert attempts[0] == 1 and attempts[1] == 1 and attempts[3] == 2 and attempts[4] == 1, attempts
    assert set(attempts) <= {1, 2}
    # errors on the path without read-backs arrive at the end of the call; the handle recovers
    bad = leaves.copy()
    bad[1, 3] = g.n
    with pytest.raises(bms.BmsError) as e:
        bms.sample_ladies(csr, torch.from_numpy(bad).cuda(), s, 7, recycle=res)
    assert e.value.code == bms.ERANGE
    res = bms.sample_ladies(csr, torch.from_numpy(hubs).cuda(), s, 8)
    res = bms.sample_ladies(csr, torch.from_numpy(hubs).cuda(), s, 9, recycle=res)
    assert_hops_equal(res.hops(), O.sample_ladies(rowptr, col, hubs, s, 9), with_p=True, what="after the error")
    # another shape on the same result: nothing remembered applies
    res = bms.sample_ladies(csr, torch.from_numpy(hubs[:2]).cuda(), s, 10, recycle=res)
    assert_hops_equal(res.hops(), O.sample_ladies(rowptr, col, hubs[:2], s, 10), with_p=True, what="other shape")


def test_shapes_around_the_window_and_part_boundaries(mods):
    # vertex counts just below, at and above one and two id windows (2^16); one seed per minibatch; one draw;
    # as many draws as the LDS path takes; recycled calls (sizes remembered) in between
    rng = np.random.default_rng(99)
    cases = [(65535, 3, 7, (5, 3)), (65536, 2, 1, (1, 1, 1)), (65537, 4, 33, (64, 1)), (131071, 1, 50, (200,)),
             (131072, 5, 20, (4096, 17)), (131073, 2, 64, (100, 100, 100)), (4097, 3, 16, (33, 9)), (70, 2, 5, (4, 4))]
    for n, k, b, s in cases:
        rowptr, col = random_csr(n, 12.0, rng)
        batches = random_batches(n, k, b, rng)
        csr, res, _ = _run_both(mods, rowptr, col, batches, s, 40 + k, mb_base=k, squared=bool(b & 1))
        O, bms, _ = mods
        for seed in (1, 2):
            res = bms.sample_ladies(csr, torch.from_numpy(batches).cuda(), s, seed, squared=bool(b & 1), recycle=res)
            assert_hops_equal(res.hops(), O.sample_ladies(rowptr, col, batches, s, seed, 0, bool(b & 1)), with_p=True,
                              what="n=%d k=%d b=%d s=%s seed=%d" % (n, k, b, s, seed))


@pytest.mark.parametrize("rows,degree,squared", [(512, 300, False), (513, 300, True), (1025, 12, False), (600, 4000, False)])
def test_windows_from_empty_to_nearly_full(mods, rows, degree, squared):
    # a wave's rows are 32 (up to 512 in all) or 64; its 4096 counters are listed at once up to 960 in use, else 32 or 8 lanes at a time:
    # no neighbours beyond id 90000, `degree` a row below 20000 (crowded: up to every counter), two a row in between
    rng = np.random.default_rng(rows + degree)
    n = 140_000
    rowptr = np.zeros(n + 1, dtype=np.int64)
    rowptr[1:rows + 1] = np.arange(1, rows + 1) * (degree + 2)
    rowptr[rows + 1:] = rowptr[rows]
    col = np.concatenate([np.concatenate([np.sort(rng.choice(20_000, degree, replace=False)),
                                          np.sort(rng.choice(70_000, 2, replace=False)) + 20_000])
                          for _ in range(rows)]).astype(np.int32)
    batches = np.stack([rng.permutation(rows), rng.permutation(rows)]).astype(np.int32)
    _run_both(mods, rowptr, col, batches, (64,), 31, squared=squared)


@pytest.mark.parametrize("s", [64, 513, 1024, 1025, 2049, 4096])
@pytest.mark.parametrize("n,degree,squared", [(12, 1, False), (40, 2, True), (60_000, 80, False)])
def test_draws_from_hardly_any_entries_to_many_blocks(mods, n, degree, squared, s):
    # 1, 2 or 4 draws per thread; P of fewer than 16 entries in all, of a few blocks of 16 that minibatches share, and of more
    # blocks than the 2048 groups the search keeps (a row of weight sums at every block's end)
    rng = np.random.default_rng(n + s)
    rowptr = np.arange(n + 1, dtype=np.int64) * degree
    col = np.concatenate([np.sort(rng.choice(n, degree, replace=False)) for _ in range(n)]).astype(np.int32)
    batches = random_batches(n, 3, min(n // 4, 900), rng)
    _run_both(mods, rowptr, col, batches, (s,), 7, mb_base=1, squared=squared)


@pytest.mark.parametrize("n,k,degree", [(200_000, 3, 30_000), (4_300_000, 2, 500), (50, 40, 3)])
def test_rows_over_many_tiles_and_windows(mods, n, k, degree):
    # rows that hold the starts of many tiles of the gathered order next to rows that hold none and empty rows; more parts of
    # windows (66 windows) than the scan has threads; minibatches smaller than a workgroup's rows
    rng = np.random.default_rng(n)
    rows = min(n // 2, 60)
    deg = np.zeros(n, dtype=np.int64)
    deg[:rows] = rng.choice([0, 1, degree // 3, degree], rows)
    deg[0] = degree
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(n, d, replace=False)) for d in deg[:rows]]).astype(np.int32)
    batches = np.stack([rng.permutation(rows)[:rows // 2] for _ in range(k)]).astype(np.int32)
    batches[:, 0] = 0
    for i in range(k):
        batches[i, 1:] = rng.permutation(np.arange(1, rows))[:rows // 2 - 1]
    _run_both(mods, rowptr, col, batches, (300,), 13, mb_base=4)


@pytest.mark.parametrize("n,degree,squared", [(40_000, 21_000, False), (2_600_000, 1_200_000, False), (4_500_000, 2_400_000, True)])
def test_draws_through_sums_of_blocks_and_groups(mods, n, degree, squared):
    # rows of P of just over 2048 blocks of 16 entries, and of over 2 and 4 million entries (groups of 2, 128 and 256 blocks in LDS,
    # the place in the group found by one and by three rounds of probes); the minibatches begin and end anywhere in a block
    rng = np.random.default_rng(n)
    rows = 6
    deg = np.zeros(n, dtype=np.int64)
    deg[:rows] = degree - np.arange(rows) * 77
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.permutation(n)[:d]) for d in deg[:rows]]).astype(np.int32)
    batches = np.array([[0, 1, 2], [3, 4, 5], [0, 3, 4]], dtype=np.int32)
    for s in ((700,), (2048,), (4096,)):
        _run_both(mods, rowptr, col, batches, s, 5, mb_base=2, squared=squared)


# 64 x 4 (minibatch, window) pairs count in 16 bits, 65 x 4 in 8; vertices that reach 8 bits' limit, pass it and wrap round to 0, in every
# place of a counter word, at the ends of both halves of a window, beside one another and alone
@pytest.mark.parametrize("squared", [False, True])
@pytest.mark.parametrize("k,b", [(64, 600), (65, 255), (65, 256), (65, 600)])
def test_counters_of_8_bits(mods, k, b, squared):
    rng = np.random.default_rng(k + b)
    n = 200_000
    rows = {255: (0, 32767, 65535, 65539), 256: (65536, 65537, 98307, 131070), 257: (98303, 98304, 131071), 512: (131074, 131075),
            600: (196607, 196608, 199999)}
    lists = []
    for t in range(b):          # neighbours of a minibatch's seed t
        lists.append([v for count, ids in rows.items() if t < count for v in ids])
    col, rowptr = [], np.zeros(n + 1, dtype=np.int64)
    for v in range(n):
        own = set(rng.integers(0, n, 2).tolist())
        if v < k * b:
            own |= set(lists[v % b])
        col.append(np.array(sorted(own), dtype=np.int32))
        rowptr[v + 1] = rowptr[v] + len(own)
    batches = np.arange(k * b, dtype=np.int32).reshape(k, b)
    _run_both(mods, rowptr, np.concatenate(col), batches, (300, 40), 7, squared=squared)


# counters of 8 bits, two parts of a window per wave: parts of 4096 counters with none to all of them in use, evenly and in one half, so
# that they are listed at once, by halves of the lanes and by 8 lanes; up to 256 rows are taken 32 at a time, more 64 at a time
@pytest.mark.parametrize("squared", [False, True])
@pytest.mark.parametrize("b", [5, 256, 257])
def test_crowded_counters_of_8_bits(mods, b, squared):
    O, bms, _ = mods
    rng = np.random.default_rng(b)
    n, k = 131_072, 130
    used = []
    for part, count in enumerate([0, 1, 500, 959, 960, 961, 1500, 1920, 1921, 2047, 2048, 2049, 3000, 3841, 4095, 4096] * 2):
        among = 4096 if part < 16 or count > 2048 else 2048      # second window: in the lower half of the part
        used.append(part * 4096 + np.sort(rng.choice(among, count, replace=False)))
    used = np.concatenate(used)
    # row 0 has all of them, where few rows make no large counters likely; many rows have most of them together
    rows = [used if b == 5 else used[::b]] + [used[rng.random(len(used)) < 2.0 / b] for _ in range(3 * b)]
    rowptr = np.zeros(n + 1, dtype=np.int64)
    rowptr[1:len(rows) + 1] = np.cumsum([len(r) for r in rows])
    rowptr[len(rows) + 1:] = rowptr[len(rows)]
    col = np.concatenate(rows).astype(np.int32)
    batches = np.stack([np.append(rng.permutation(3 * b)[:b - 1] + 1, 0) for _ in range(k)]).astype(np.int32)
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as profile:
        _run_both(mods, rowptr, col, batches, (200,), 5, squared=squared)
        torch.cuda.synchronize()
    names = [e.name for e in profile.events() if "ldw_accumulate_kernel" in e.name]
    assert len(names) == 2 and all("<%s, true>" % str(squared).lower() in x for x in names), names


# more than 2048 (minibatch, window) pairs: the copy of P by parts, which begin anywhere in a memory line and hold from no entry to a
# few hundred; 512 workgroups take several pairs each, some of which are counted by halves (b = 300)
@pytest.mark.parametrize("squared", [False, True])
@pytest.mark.parametrize("k,b,shared", [(520, 250, 60), (520, 300, 60), (513, 40, 0), (693, 17, 5)])
def test_many_pairs(mods, k, b, shared, squared):
    O, bms, _ = mods
    rng = np.random.default_rng(k + b)
    n = 200_000
    common = rng.choice(n, shared, replace=False)
    rows = [np.unique(np.concatenate([common, rng.integers(0, n, int(rng.integers(0, 120)))])) for _ in range(3 * b)]
    lengths = np.full(n, 3)             # (so that the graph has the columns for an index)
    lengths[:len(rows)] = [len(r) for r in rows]
    rowptr = np.concatenate([[0], np.cumsum(lengths)])
    rest = np.sort(rng.integers(0, n // 3, (n - len(rows), 3)) + np.arange(3) * (n // 3), axis=1)
    col = np.concatenate(rows + [rest.ravel()]).astype(np.int32)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    for index in (False, True):         # the rows' lists found by the hop, or taken from the index beside the rows
        res = None
        for call in range(2):           # the first call of a shape and a recycled one
            batches = np.stack([rng.permutation(3 * b)[:b] for _ in range(k)]).astype(np.int32)
            ref = O.sample_ladies(rowptr, col, batches, (50,), 11 + call, 0, squared)
            with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as profile:
                res = bms.sample_ladies(csr, torch.from_numpy(batches).cuda(), (50,), 11 + call, squared=squared, recycle=res, index=index)
                torch.cuda.synchronize()
            names = " ".join(e.name for e in profile.events())
            assert "ldw_win_scan_kernel" in names and "ldw_p_copy_kernel" in names
            assert call == 0 or ("ldw_bounds_transpose_kernel" in names) != index, names
            assert_hops_equal(res.hops(), ref, with_p=True, what="index %s call %d" % (index, call))


# more than 2048 pairs with counters of 8 bits: parts from 256 columns on are staged as a bit per column and a byte per entry.  Parts of
# 4096 columns with none to all of them in use, evenly and in their lower half: listed at once, by halves of the lanes and by 8 lanes on
# the way out, whose words of four bytes then begin in one listing and end in the next; at once or by halves (2048) on the way back
@pytest.mark.parametrize("squared", [False, True])
@pytest.mark.parametrize("b", [5, 257])
def test_parts_as_masks(mods, b, squared):
    O, bms, _ = mods
    rng = np.random.default_rng(b)
    n, k = 131_072, 1025
    used = []
    for part, count in enumerate([0, 1, 255, 256, 257, 955, 956, 957, 1500, 1911, 1913, 2047, 2048, 2049, 3000, 4096] * 2):
        among = 4096 if part < 16 or count > 2048 else 2048      # second window: in the lower half of the part
        used.append(part * 4096 + np.sort(rng.choice(among, count, replace=False)))
    used = np.concatenate(used)
    rows = [used if b == 5 else used[::b]] + [used[rng.random(len(used)) < 2.0 / b] for _ in range(3 * b)]
    rowptr = np.zeros(n + 1, dtype=np.int64)
    rowptr[1:len(rows) + 1] = np.cumsum([len(r) for r in rows])
    rowptr[len(rows) + 1:] = rowptr[len(rows)]
    col = np.concatenate(rows).astype(np.int32)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = None
    for call in range(2):
        batches = np.stack([np.append(rng.permutation(3 * b)[:b - 1] + 1, 0) for _ in range(k)]).astype(np.int32)
        ref = O.sample_ladies(rowptr, col, batches, (200,), 5, 0, squared)
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as profile:
            res = bms.sample_ladies(csr, torch.from_numpy(batches).cuda(), (200,), 5, squared=squared, recycle=res)
            torch.cuda.synchronize()
        names = " ".join(e.name for e in profile.events())
        assert "ldw_accumulate_kernel<%s, true>" % str(squared).lower() in names and "ldw_p_copy_kernel" in names, names
        assert_hops_equal(res.hops(), ref, with_p=True, what="call %d" % call)


# parts as masks from 256 entries a part on, by what P had in the call before: long and short parts where the other kind was likely
@pytest.mark.parametrize("squared", [False, True])
def test_masks_by_the_entries_of_a_part(mods, squared):
    O, bms, _ = mods
    rng = np.random.default_rng(77)
    n, k, b = 131_072, 1025, 20
    lengths = np.zeros(n, dtype=np.int64)
    lengths[:2000], lengths[2000:4000] = 600, 30
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(n, x, replace=False)) for x in lengths[:4000]]).astype(np.int32)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = None
    for call, (first, masks) in enumerate([(0, True), (0, True), (2000, True), (2000, False), (0, True), (0, True)]):
        batches = np.stack([first + rng.permutation(2000)[:b] for _ in range(k)]).astype(np.int32)
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as profile:
            res = bms.sample_ladies(csr, torch.from_numpy(batches).cuda(), (40,), 9 + call, squared=squared, recycle=res)
            torch.cuda.synchronize()
        for kernel in ("ldw_accumulate_kernel", "ldw_p_copy_kernel"):       # (the last attempt's)
            name = [e.name for e in profile.events() if kernel in e.name][-1]
            assert ("LwMasks" in name) == masks, (call, name)
        assert res.attempts() == (2 if call == 4 else 1)
        assert_hops_equal(res.hops(), O.sample_ladies(rowptr, col, batches, (40,), 9 + call, 0, squared), with_p=True, what="call %d" % call)


# the draws of a minibatch by one workgroup and by two, four and eight, which count one another in every call anew; some minibatches have
# no neighbours to draw from, and P of the third call is more than what was provided for it, so that there are no draws
@pytest.mark.parametrize("k,s", [(128, 1023), (128, 1024), (129, 1024), (64, 2049), (3, 4095), (31, 4096)])
def test_draws_by_several_workgroups(mods, k, s):
    O, bms, _ = mods
    rng = np.random.default_rng(s + k)
    n, b = 30_000, 20
    lengths = np.concatenate([np.zeros(b, dtype=np.int64), rng.integers(20, 60, 10_000), np.full(n - 10_000 - b, 400)])
    lengths[12_000:] = 0
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(n, x, replace=False)) for x in lengths]).astype(np.int32)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = None
    for call in range(4):
        ids = np.arange(10_000 + b, 12_000) if call == 2 else np.arange(b, 10_000)
        batches = np.stack([rng.permutation(ids)[:b] for _ in range(k)]).astype(np.int32)
        batches[k // 2] = np.arange(b)
        res = bms.sample_ladies(csr, torch.from_numpy(batches).cuda(), (s, 7), 3 + call, recycle=res)
        assert_hops_equal(res.hops(), O.sample_ladies(rowptr, col, batches, (s, 7), 3 + call), with_p=True, what="call %d" % call)
        assert res.attempts() == (2 if call == 2 else 1)


# lists of window boundaries in one piece and in several (up to 64 boundaries each, of many rows up to 128); rows that fill no tile of 64
@pytest.mark.parametrize("windows,k", [(1, 5), (2, 5), (62, 5), (63, 5), (64, 5), (126, 5), (127, 5), (128, 5), (63, 1800), (126, 900),
                                       (127, 900), (128, 900), (255, 500), (256, 500)])
def test_lists_of_boundaries_in_pieces(mods, windows, k):
    O, bms, _ = mods
    rng = np.random.default_rng(windows)
    n = windows * 65536 - 7
    lengths = np.zeros(n, dtype=np.int64)
    some = np.unique(np.concatenate([rng.integers(0, n, 400), [0, n - 1]]))
    lengths[some] = rng.integers(0, 90, len(some))
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(some, x, replace=False)) for x in lengths[some]]).astype(np.int32)
    batches = np.stack([rng.permutation(some)[:37] for _ in range(k)]).astype(np.int32)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    ref = O.sample_ladies(rowptr, col, batches, (50, 20), 7)
    res = None
    for call in range(2):
        res = bms.sample_ladies(csr, torch.from_numpy(batches).cuda(), (50, 20), 7, recycle=res)
        assert_hops_equal(res.hops(), ref, with_p=True, what="%d windows, call %d" % (windows, call))


# more parts than a launch of the copy of P has waves
def test_more_pairs_than_workgroups_copy(mods):
    O, bms, _ = mods
    rng = np.random.default_rng(8)
    n, k = 100_000, 33_000
    rowptr, col = random_csr(n, 20.0, rng)
    batches = random_batches(n, k, 2, rng)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = bms.sample_ladies(csr, torch.from_numpy(batches).cuda(), (5,), 3)
    assert_hops_equal(res.hops(), O.sample_ladies(rowptr, col, batches, (5,), 3), with_p=True, what="k=%d" % k)


# seeds that lie in the result's own rows when the first kernel reads them: copied there from the host, or the rows of the call before
@pytest.mark.parametrize("k,b", [(3, 300), (9, 64), (2, 4096)])
def test_seeds_in_the_rows_of_the_result(mods, k, b):
    O, bms, _ = mods
    rng = np.random.default_rng(b)
    rowptr, col = random_csr(100_000, 9.0, rng)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    batches = random_batches(100_000, k, b, rng)
    seeds, res = batches, None
    for call in range(4):
        res = bms.sample_ladies(csr, seeds, (40, 20), 3 + call, recycle=res)
        assert_hops_equal(res.hops(), O.sample_ladies(rowptr, col, batches, (40, 20), 3 + call), with_p=True, what="call %d" % call)
        rows = res.hop(0).row_vertex
        seeds = rows.view(k, b) if call else batches


# P of 10 million entries and more is stored past the caches, a smaller one, which the draws then find there, is not, whatever the number
# of (minibatch, window) pairs; in the first call, where a bound of its size decides, and in recycled ones
@pytest.mark.parametrize("squared", [False, True])
@pytest.mark.parametrize("k,b,past", [(520, 40, False), (640, 460, True)])
def test_large_p_past_the_caches(mods, k, b, past, squared):
    O, bms, _ = mods
    rng = np.random.default_rng(k)
    n = 200_000
    rowptr, col = random_csr(n, 50.0, rng)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = None
    for call in range(2):
        batches = random_batches(n, k, b, rng)
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as profile:
            res = bms.sample_ladies(csr, torch.from_numpy(batches).cuda(), (30,), 17 + call, squared=squared, recycle=res)
            torch.cuda.synchronize()
        name, = [e.name for e in profile.events() if "ldw_p_copy_kernel" in e.name]
        assert "<%s, %s>" % (str(squared).lower(), str(past).lower()) in name, name
        assert (res.hop(0).pnnz >= 10_000_000) == past
        assert_hops_equal(res.hops(), O.sample_ladies(rowptr, col, batches, (30,), 17 + call, 0, squared), with_p=True, what="call %d" % call)


# the call's sizes and the minibatches' offsets left for the host by the last kernel, or, of more than 512 offsets, by a launch of its
# own (that there are no offsets for the host any more is the case of 22000 minibatches)
@pytest.mark.parametrize("k,b,s,own", [(511, 3, (5,), False), (512, 3, (5,), True), (169, 4, (6, 5, 4), False), (170, 4, (6, 5, 4), True),
                                       (7000, 2, (2, 2, 3), True), (22_000, 1, (1,), False)])
def test_offsets_left_for_the_host(mods, k, b, s, own):
    O, bms, _ = mods
    rng = np.random.default_rng(k)
    rowptr, col = random_csr(3000, 6.0, rng)
    csr = bms.Csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    res = None
    for call in range(3):
        batches = random_batches(3000, k, b, rng)
        ref = O.sample_ladies(rowptr, col, batches, s, 21 + call)
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as profile:
            res = bms.sample_ladies(csr, torch.from_numpy(batches).cuda(), s, 21 + call, recycle=res)
            torch.cuda.synchronize()
        assert any("publish_kernel" in e.name for e in profile.events()) == own
        assert_hops_equal(res.hops(), ref, with_p=True, what="call %d" % call)
        for hop, want in enumerate(ref):
            for i in (0, 1, k // 2, k - 2, k - 1):
                m = res.minibatch(hop, i)
                r0, r1, c0, c1 = want.mb_rowoff[i], want.mb_rowoff[i + 1], want.mb_coloff[i], want.mb_coloff[i + 1]
                assert (m.row0, m.rows, m.col0, m.ncols) == (r0, r1 - r0, c0, c1 - c0)
                assert (m.edge0, m.nnz) == (want.rowptr[r0], want.rowptr[r1] - want.rowptr[r0])
