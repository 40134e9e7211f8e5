"""How a large feature fetch divides its ids (csrc/feature_runs.h, run on the host): minibatches are found, every row is in a
tile, and ids of any other order cost little more than their rows."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("feature_runs") / "feature_runs_host.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall",
                           "-I", os.path.join(ROOT, "paper_2311_02909_amd", "csrc"), "-o", so,
                           os.path.join(ROOT, "tests", "host", "feature_runs_host.cpp")])
    lib = C.CDLL(so)
    for f in (lib.replay, lib.probe, lib.sample):
        f.restype = C.c_int64
    return lib


def _replay(lib, ids):
    """runs found, the longest tile, distance of the tiles' first ids (the tiles of every run follow one another)"""
    ids = np.ascontiguousarray(ids, dtype=np.int32)
    longest, apart = C.c_int64(), C.c_int64()
    runs = lib.replay(ids.ctypes.data_as(C.c_void_p), C.c_int64(len(ids)), C.byref(longest), C.byref(apart))
    assert runs > 0
    return runs, longest.value, apart.value


def _stack(rng, n, lengths):
    return np.concatenate([np.sort(rng.choice(n, size=x, replace=False)) for x in lengths])


def test_probes_lie_between_their_samples(lib):
    for m in (64 * 1024, 65_537, 1_000_003, 40_000_000_000):
        m = C.c_int64(m)
        for s in range(1023):
            assert lib.sample(s, m) < lib.probe(s, m) < lib.sample(s + 1, m)


@pytest.mark.parametrize("k,m,n", [(2, 70_000, 100_000), (16, 400_000, 60_000), (32, 4_000_000, 1_000_000), (256, 1_000_000, 9000),
                                   (400, 1_000_000, 500_000), (512, 1_050_000, 30_000), (2, 1_200_000, 5_000_000)])
def test_minibatches_are_found(lib, k, m, n):
    rng = np.random.default_rng(k)
    lengths = rng.integers(int(0.8 * m / k), int(1.2 * m / k) + 1, size=k)
    runs, longest, apart = _replay(lib, _stack(rng, n, lengths))
    assert 0.95 * k <= runs <= k
    # tiles of about 128 rows that start at the same ids (but the first ones of a run) up to the gap between two ids
    assert longest < 512 and apart < 40 * n * k / m


def _orders(rng, m):
    n = 10 * m
    yield "shuffled", lambda: rng.integers(0, n, size=m)
    yield "descending", lambda: np.arange(m)[::-1]
    yield "all the same", lambda: np.full(m, 7)
    for length in (5, 64, 1000, m // 1023, m // 512, m // 900, m // 1500, m // 3000):   # runs too short to be found
        yield "runs of %d" % length, lambda: np.concatenate(
            [np.sort(rng.integers(0, n, size=min(length, m - x))) for x in range(0, m, length)])
        yield "equal runs of %d" % length, lambda: np.arange(m) % length
    for share in (0.01, 0.1, 0.3):
        def mixed():
            ids = _stack(rng, n, [m // 8] * 8)
            at = rng.random(len(ids)) < share
            ids[at] = rng.integers(0, n, size=int(at.sum()))
            return ids
        yield "%g of the ids of 8 minibatches at random" % share, mixed
    yield "shuffled in blocks", lambda: np.sort(rng.integers(0, n, size=(8, m // 8)), axis=1).reshape(8, -1, 50)[
        :, :, rng.permutation(50)].reshape(-1) if m % 400 == 0 else np.arange(m)

    def part():
        ids = np.sort(rng.integers(0, n, size=(40, m // 40)), axis=1)
        ids[:3] = rng.integers(0, n, size=ids[:3].shape)
        return ids.reshape(-1)
    yield "three of forty minibatches shuffled", part

    def first():
        ids = np.sort(rng.integers(0, n, size=(40, m // 40)), axis=1)
        ids[0] = rng.permutation(ids[0])
        return ids.reshape(-1)
    yield "the first of forty minibatches shuffled", first


@pytest.mark.parametrize("m", [66_000, 262_000, 1_000_000, 4_000_000])
def test_any_other_order(lib, m):
    # every row in one tile, and no tile much longer than others.  By the samples' descents alone every second draw of unordered
    # ids passes for minibatches, and tiles found one by one lay across each other: 7 times the rows at 10 million
    rng = np.random.default_rng(m)
    for name, make in _orders(rng, m):
        for draw in range(8 if name == "shuffled" else 1):
            runs, longest, _ = _replay(lib, make())
            if name == "shuffled":
                assert runs == 1 and longest == 128, name
            assert longest <= 129 + 2 * max(4096, m // 16), (name, runs, longest)
