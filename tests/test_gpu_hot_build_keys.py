"""Build sides with frequent keys: LDS tables whose entries spread over many buckets behind their
own (walked by one lane and by the whole wave), alone and among other keys that share them,
against counts and lookups in torch."""
import pytest
import torch

from tests.gpu_util import gpu, log, need_gpu


def _join(rk, sk, bits, deterministic=False):
    from paper_1904_11201_amd import _native
    from paper_1904_11201_amd import join as J
    _native.tune_set("hash.bits", bits, local=True)
    _native.tune_set("hash.deterministic", int(deterministic), local=True)
    try:
        return J.hash_join(J.Relation(rk), J.Relation(sk))
    finally:
        _native.tune_set("hash.bits", None, local=True)
        _native.tune_set("hash.deterministic", None, local=True)


def _check(rk, sk, pairs):
    """Each pair joins equal keys, no pair occurs twice, and their number is exact."""
    counts = torch.bincount((rk - rk.min()).long())
    at = (sk - rk.min()).long()
    inside = (at >= 0) & (at < counts.numel())
    assert pairs.shape[0] == int(counts[at[inside]].sum())
    assert torch.equal(rk[pairs[:, 0].long()], sk[pairs[:, 1].long()])
    packed = pairs.view(torch.int64).reshape(-1)
    assert packed.unique().numel() == packed.numel()


@gpu
@pytest.mark.parametrize("bits", [0, 1, 6])
@pytest.mark.parametrize("copies", [5, 9, 64, 65, 66, 72, 600, 5000, 20000])
def test_one_frequent_key_among_others(bits, copies):
    need_gpu()
    g = torch.Generator(device="cuda")
    g.manual_seed(copies)
    rk = torch.randint(0, 6000, (9000,), device="cuda", dtype=torch.int32, generator=g)
    rk = torch.cat([rk, torch.full((copies,), 777, device="cuda", dtype=torch.int32)])
    rk = rk[torch.randperm(rk.numel(), device="cuda", generator=g)]
    sk = torch.randperm(7000, device="cuda", generator=g).to(torch.int32)
    log(f"frequent key, {copies} copies, bits {bits}")
    _check(rk, sk, _join(rk, sk, bits))


@gpu
@pytest.mark.parametrize("deterministic", [False, True])
def test_zipf_build_side(deterministic):
    need_gpu()
    n = 60_000
    g = torch.Generator(device="cuda")
    g.manual_seed(8)
    u = torch.rand(n, device="cuda", generator=g, dtype=torch.float64)
    rk = (torch.exp(u * 9.0).to(torch.int32) * 7919) % 8000
    sk = torch.randperm(8000, device="cuda", generator=g).to(torch.int32)
    log(f"Zipf build side, deterministic {deterministic}")
    pairs = _join(rk, sk, 5, deterministic)
    _check(rk, sk, pairs)
    if deterministic:
        assert torch.equal(pairs, _join(rk, sk, 5, deterministic))


@gpu
def test_every_row_the_same_key():
    need_gpu()
    rk = torch.full((10_000,), -5, device="cuda", dtype=torch.int32)
    sk = torch.tensor([-5, 3, -5, -6], device="cuda", dtype=torch.int32)
    for bits in (0, 2, 7):
        log(f"one key, bits {bits}")
        _check(rk, sk, _join(rk, sk, bits))
