"""The rule that picks the unpartitioned or the partitioned path for a small build side, on both
sides of its line, against the same join with the path forced by the "hash.single_max_chunks" knob."""
import pytest
import torch

from tests.gpu_util import gpu, log, need_gpu

LINE = 6 << 20  # repeated probes, (R chunks - 1) * |S|, from which a join is partitioned
CAP = 9216


def _relations(nR, nS, seed, rids):
    from paper_1904_11201_amd import join as J
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rk = torch.randperm(nR, device="cuda", generator=g).to(torch.int32)
    rk[nR // 2:nR // 2 + nR // 8] = rk[:nR // 8]  # some keys twice
    sk = torch.randint(-5, nR, (nS,), device="cuda", dtype=torch.int32, generator=g)
    rr = torch.randperm(nR, device="cuda", generator=g).to(torch.int32) if rids else None
    return J.Relation(rk, rid=rr), J.Relation(sk)


def _sorted(pairs):
    return pairs.view(torch.int64).reshape(-1).sort().values


@gpu
@pytest.mark.parametrize("nR", [CAP, CAP + 1, 36_000, 16 * CAP, 16 * CAP + 1])
@pytest.mark.parametrize("side", ["below", "above"])
def test_both_sides_of_the_line(nR, side):
    from paper_1904_11201_amd import _native
    from paper_1904_11201_amd import join as J
    need_gpu()
    repeats = max(1, -(-nR // CAP) - 1)
    nS = LINE // repeats + (0 if side == "below" else 1)
    R, S = _relations(nR, nS, nR, rids=side == "above")
    log(f"plan rule {nR} x {nS} ({side} the line)")
    got = _sorted(J.hash_join(R, S))
    try:
        for chunks in (0, 17):  # partitioned, unpartitioned
            _native.tune_set("hash.single_max_chunks", chunks, local=True)
            assert torch.equal(got, _sorted(J.hash_join(R, S))), chunks
    finally:
        _native.tune_set("hash.single_max_chunks", None, local=True)


@gpu
def test_noalloc_keeps_small_builds_with_many_probe_rows():
    """The partitioned form of this join does not fit the 64 MiB scratch array; it is joined
    unpartitioned there."""
    from paper_1904_11201_amd import join as J
    need_gpu()
    R, S = _relations(20_000, 9_000_000, 3, rids=False)
    assert J.join_workspace_bytes(J.JOIN_KIND_HASH, R.n, S.n) > 64 << 20
    log("noalloc 20000 x 9000000")
    want = _sorted(J.hash_join(R, S))
    out = torch.empty((want.numel(), 2), dtype=torch.int32, device="cuda")
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    J.join_hash_noalloc(R, S, out, count)
    assert int(count[0]) == want.numel() and torch.equal(_sorted(out), want)


@gpu
@pytest.mark.parametrize("nS", [1024, 65 * 1024, 128 * 1024, 128 * 1024 + 1, 130 * 1024])
def test_unit_counts_published_or_scanned(nS):
    """One probe unit per 1024 rows: up to 128 units publish their counts themselves, more are
    scanned; a second write from the same count, into a larger output, gives the same pairs."""
    from paper_1904_11201_amd import join as J
    need_gpu()
    R, S = _relations(3000, nS, nS, rids=True)
    log(f"unit counts 3000 x {nS}")
    ws = J.workspace(J.JOIN_KIND_HASH, R.n, S.n)
    n = J.join_count(J.JOIN_KIND_HASH, R, S, None, ws)
    out = torch.full((n + 5, 2), -9, dtype=torch.int32, device="cuda")
    with pytest.raises(J.JoinError):
        J.join_materialize(J.JOIN_KIND_HASH, R, S, None, ws, out[:n - 1])
    J.join_materialize(J.JOIN_KIND_HASH, R, S, None, ws, out)
    assert bool((out[n:] == -9).all())
    pairs = torch.empty((n, 2), dtype=torch.int32, device="cuda")
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    J.join_hash_noalloc(R, S, pairs, count)  # always scanned
    assert int(count[0]) == n and torch.equal(out[:n], pairs)
