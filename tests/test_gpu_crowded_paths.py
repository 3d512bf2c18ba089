"""Hot build keys (hundreds of copies in one LDS table, so the unit is joined by sorted entries)
through each way into the hash join, against the oracle's pairs."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_1904_11201_amd import datagen
from tests.gpu_util import canon_gpu, dev_rel, gpu, log, need_gpu


def _key_of_hash(h):
    """The int32 key whose hash (common.hpp hmix) is h: the finaliser's steps undone in turn."""
    m = 0xFFFFFFFF
    h ^= h >> 16
    h = h * pow(0xC2B2AE35, -1, 1 << 32) & m
    h ^= h >> 13 ^ h >> 26
    h = h * pow(0x85EBCA6B, -1, 1 << 32) & m
    h ^= h >> 16
    return h - (1 << 32) if h >= 1 << 31 else h


# a key of each pair of top hash bits (the partition's, which an empty slot's marker is made from),
# and the one whose hash is the marker of a table made from hash 0
HOT = [2, 1, 3, 5, _key_of_hash(0x80000000)]


def _hot_join(hot, nR, nS, copies, seed=91, domain=10_000_000):
    """R: nR uniform keys and `copies` rows of each hot key; S: nS uniform keys and 40 of each."""
    g = datagen.rng_for(seed)
    rk = np.concatenate([datagen.uniform_keys(g, nR, 0, domain), np.repeat(np.array(hot, np.int32), copies)])
    sk = np.concatenate([datagen.uniform_keys(g, nS, 0, domain), np.repeat(np.array(hot, np.int32), 40)])
    R = datagen.Rel(key=g.permutation(rk).astype(np.int32), rid=g.permutation(len(rk)).astype(np.int32))
    return R, datagen.Rel(key=g.permutation(sk).astype(np.int32), rid=g.permutation(len(sk)).astype(np.int32))


def _expect(R, S):
    n, ref = oracle.equi_sortmerge(R.key, S.key, Rrid=R.rid, Srid=S.rid)
    assert len(ref) == n
    return ref


@gpu
@pytest.mark.parametrize("hot,copies", [([k], 1000) for k in HOT] + [(HOT, 300), (HOT, 1000)])
def test_semi_join_of_a_hot_build_key(hot, copies):
    """More than 2^21 probe rows, so the count pass records the matching ones, in partitions of one
    chunk: the record covers the crowded units, which another kernel writes."""
    need_gpu()
    from paper_1904_11201_amd.join import hash_join
    R, S = _hot_join(hot, 200_000, (1 << 21) + 1001, copies)
    ref = _expect(R, S)
    dR, dS = dev_rel(R), dev_rel(S)
    log(f"semi-join, hot keys {hot}, {copies} copies each")
    got = canon_gpu(hash_join(dR, dS, prefilter=True))
    assert np.array_equal(got, ref)
    assert np.array_equal(canon_gpu(hash_join(dR, dS)), ref)


@gpu
@pytest.mark.parametrize("nS", [3000, 200_000, 4_000_000])
@pytest.mark.parametrize("keys,copies", [(1, 70), (1, 300), (1, 700), (3, 550), (10, 250), (40, 60), (40, 150)])
def test_around_the_line_between_walks_and_sorts(keys, copies, nS):
    """Tables with keys of about as many copies as make a unit crowded, unpartitioned and in
    partitions of one chunk, with one round of probes and many."""
    need_gpu()
    from paper_1904_11201_amd import _native
    from paper_1904_11201_amd.join import hash_join
    R, S = _hot_join(list(range(keys)), 9000 - keys * copies, nS, copies, domain=30_000)
    ref = _expect(R, S)
    dR, dS = dev_rel(R), dev_rel(S)
    for bits in (0, 1):
        _native.tune_set("hash.bits", bits, local=True)
        try:
            log(f"crowd line, {keys} keys of {copies}, {nS} probes, bits {bits}")
            assert np.array_equal(canon_gpu(hash_join(dR, dS)), ref)
        finally:
            _native.tune_set("hash.bits", None, local=True)


@gpu
def test_moderately_hot_keys_are_walked():
    """9000 x 10,000 with one key of 160 copies that no row asks for: at most 4 times the join without
    it (sorting its tables took 8 times, their walks 2)."""
    need_gpu()
    import time

    import torch

    from paper_1904_11201_amd.join import hash_join
    took = {}
    for copies in (1, 160):
        R, S = _hot_join([7], 9000 - copies, 10_000, copies, domain=1_000_000)
        S.key[S.key == 7] = 8
        R, S = dev_rel(R), dev_rel(S)
        log(f"one key of {copies} copies")
        runs = []
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            hash_join(R, S)
            torch.cuda.synchronize()
            runs.append(time.perf_counter() - t0)
        took[copies] = min(runs)
    log(f"us: {[(k, round(v * 1e6)) for k, v in took.items()]}")
    assert took[160] < 4 * took[1]


def _noalloc(R, S, cap):
    import ctypes

    import torch

    from paper_1904_11201_amd import _native
    pairs = torch.empty((cap, 2), dtype=torch.int32, device="cuda")
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    rr, sr = R.c(), S.c()
    rc = _native.lib.join_hash_noalloc(ctypes.byref(rr), ctypes.byref(sr), ctypes.c_void_p(pairs.data_ptr()), cap,
                                       ctypes.c_void_p(count.data_ptr()), None)
    assert rc == _native.JOIN_OK, _native.last_error()
    assert int(count.item()) == cap
    return pairs


def _written_by_another_thread(R, S, n):
    """The count pass on this thread, the write pass on one that knows nothing of it."""
    import threading

    import torch

    from paper_1904_11201_amd import join as J
    ws = J.workspace(J.JOIN_KIND_HASH, R.n, S.n)
    assert J.join_count(J.JOIN_KIND_HASH, R, S, None, ws) == n
    pairs, errors = torch.empty((n, 2), dtype=torch.int32, device="cuda"), []

    def write():
        try:
            J.join_materialize(J.JOIN_KIND_HASH, R, S, None, ws, pairs)
            torch.cuda.synchronize()
        except Exception as e:  # shown by the assertion below
            errors.append(e)

    t = threading.Thread(target=write)
    t.start()
    t.join()
    assert not errors, errors
    return pairs


@gpu
@pytest.mark.parametrize("nR,copies", [(3000, 1000), (7000, 1000), (7000, 100), (200_000, 1000)])
def test_every_entry_of_a_hot_build_key(nR, copies):
    """Unpartitioned and partitioned, for tables crowded by the build and units sorted for a probe's
    long run."""
    need_gpu()
    from paper_1904_11201_amd import join as J
    R, S = _hot_join(HOT, nR, 50_000, copies, domain=60_000)
    ref = _expect(R, S)
    dR, dS = dev_rel(R), dev_rel(S)
    for name, run in (("resident build", lambda: J.ResidentBuild(dR).probe(dS)),
                      ("noalloc", lambda: _noalloc(dR, dS, len(ref))),
                      ("written by another thread", lambda: _written_by_another_thread(dR, dS, len(ref))),
                      ("pre-filtered", lambda: J.hash_join(dR, dS, prefilter=True))):
        log(f"hot build keys, {nR} rows and {copies} copies: {name}")
        assert np.array_equal(canon_gpu(run()), ref), name


@gpu
@pytest.mark.parametrize("copies", [100, 1000])
def test_batch_with_hot_build_keys(copies):
    """Fan-outs of 0 and 1 bits (raw and unmarked tables) and more, hot jobs among others; written
    twice from one count."""
    need_gpu()
    import torch

    from paper_1904_11201_amd import join as J
    jobs, refs = [], []
    for i, (bits, hot) in enumerate([(0, HOT[:2]), (1, HOT), (-1, []), (2, HOT), (5, HOT), (-1, HOT), (0, [])]):
        R, S = _hot_join(hot, 2000 if bits == 0 else 9000, 6000 + i, copies, seed=i, domain=20_000)
        refs.append(_expect(R, S))
        jobs.append(J.Job(dev_rel(R), dev_rel(S), bits))
    log(f"batch with hot build keys, {copies} copies")
    batch = J.Batch(jobs)
    offs = batch.count().cpu().tolist()
    pairs = torch.empty((offs[-1], 2), dtype=torch.int32, device="cuda")
    for _ in range(2):
        pairs.fill_(-1)
        batch.materialize(pairs)
        for j, ref in enumerate(refs):
            assert np.array_equal(canon_gpu(pairs[offs[j]:offs[j + 1]]), ref), j


@gpu
@pytest.mark.parametrize("rows", [15, 16, 17, 127, 128, 129])
@pytest.mark.parametrize("copies", [9, 30])
def test_around_the_line_for_runs_of_matches(copies, rows):
    """`rows` probe rows, one to a thread, that match more than eight build rows each: below and above the
    counts from which a unit, or every unit of a join, is written from sorted entries."""
    need_gpu()
    from paper_1904_11201_amd import _native
    from paper_1904_11201_amd import join as J
    R, S = _hot_join([1, 2, 3], 5000, 900, copies, domain=30_000)
    S.key[:] = np.arange(len(S.key)) + 100_000
    S.key[:rows] = 1 + np.arange(rows) % 3
    ref = _expect(R, S)
    assert len(ref) >= rows * copies
    dR, dS = dev_rel(R), dev_rel(S)
    for bits in (0, 1, 3):
        _native.tune_set("hash.bits", bits, local=True)
        try:
            log(f"{rows} rows with runs of {copies}, bits {bits}")
            assert np.array_equal(canon_gpu(J.hash_join(dR, dS)), ref)
            assert np.array_equal(canon_gpu(_written_by_another_thread(dR, dS, len(ref))), ref)
            assert np.array_equal(canon_gpu(_batch(dR, dS, bits)), ref)
        finally:
            _native.tune_set("hash.bits", None, local=True)


def _batch(R, S, bits):
    import torch

    from paper_1904_11201_amd import join as J
    batch = J.Batch([J.Job(R, S, bits)])
    offs = batch.count().cpu().tolist()
    pairs = torch.empty((offs[-1], 2), dtype=torch.int32, device="cuda")
    batch.materialize(pairs)
    return pairs


def _repeated(nR, d, nS, seed=5):
    g = datagen.rng_for(seed)
    k = nR // d
    R = datagen.Rel(key=datagen.uniform_keys(g, nR, 0, k), rid=g.permutation(nR).astype(np.int32))
    return R, datagen.Rel(key=datagen.uniform_keys(g, nS, 0, 2 * k), rid=g.permutation(nS).astype(np.int32))


@gpu
@pytest.mark.parametrize("nR,nS,d", [(nR, nS, d) for d in (3, 4, 6, 12, 40)
                                     for nR, nS in ((700, 700), (9001, 2000), (30_000, 5000), (300_001, 40_000),
                                                    (2_500_000, 50_000))] +
                                    [(150_000, 2_200_000, d) for d in (3, 4, 6)])
def test_builds_of_evenly_repeated_keys(nR, nS, d):
    """Every key has about d copies: units on both sides of the lines, of one and of several rounds of
    workgroups, and joins all of whose units are sorted."""
    need_gpu()
    from paper_1904_11201_amd import join as J
    R, S = _repeated(nR, d, nS)
    ref = _expect(R, S)
    dR, dS = dev_rel(R), dev_rel(S)
    for name, run in (("join", lambda: J.hash_join(dR, dS)),
                      ("resident build", lambda: J.ResidentBuild(dR).probe(dS)),
                      ("written by another thread", lambda: _written_by_another_thread(dR, dS, len(ref))),
                      ("pre-filtered", lambda: J.hash_join(dR, dS, prefilter=True)),
                      ("batch", lambda: _batch(dR, dS, -1))):
        log(f"{nR} rows of keys with {d} copies x {nS}: {name}")
        assert np.array_equal(canon_gpu(run()), ref), name


@gpu
@pytest.mark.parametrize("nR", [9000, 400_000])
def test_evenly_repeated_keys_are_not_walked(nR):
    """Keys of 32 copies, each asked for once: at most 4 times the join of as many rows in keys of 2 (their
    walks took 10 times)."""
    need_gpu()
    import time

    import torch

    from paper_1904_11201_amd.join import hash_join
    took = {}
    for d in (2, 32):
        R, _ = _repeated(nR, d, 1)
        S = datagen.Rel(key=np.arange(nR // d, dtype=np.int32), rid=np.arange(nR // d, dtype=np.int32))
        R, S = dev_rel(R), dev_rel(S)
        log(f"{nR} rows of keys with {d} copies")
        runs = []
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            hash_join(R, S)
            torch.cuda.synchronize()
            runs.append(time.perf_counter() - t0)
        took[d] = min(runs)
    log(f"us: {[(k, round(v * 1e6)) for k, v in took.items()]}")
    assert took[32] < 4 * took[2]
