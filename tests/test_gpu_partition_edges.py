"""The histogram's and the scatter's cases: every number of LDS counters per partition (forced
fan-outs), the two tile sizes, columns at every alignment of 4 bytes, and chunk lengths around
whole rounds and odd ends, against a lookup in torch."""
import pytest
import torch

from tests.gpu_util import gpu, log, need_gpu


def _lookup(one, many):
    keys, order = one.long().sort()
    at = torch.searchsorted(keys, many.long()).clamp_(max=keys.numel() - 1)
    return torch.where(keys[at] == many.long(), order[at], torch.full_like(at, -1))


@gpu
@pytest.mark.parametrize("bits", [1, 4, 5, 6, 9, 10, 11])
@pytest.mark.parametrize("nR,nS", [(5000, 4099), (40_000, 16384 * 3 + 4095), (9, 300_001)])
def test_fan_outs_and_alignments(bits, nR, nS):
    from paper_1904_11201_amd import _native
    from paper_1904_11201_amd import join as J
    need_gpu()
    g = torch.Generator(device="cuda")
    g.manual_seed(bits * 1000 + nR)
    for shift in range(4):
        one = torch.randperm(nR, device="cuda", generator=g).to(torch.int32)
        many = torch.randint(-3, nR + 3, (nS + shift,), device="cuda", dtype=torch.int32, generator=g)[shift:]
        rid = torch.arange(nS + 1, device="cuda", dtype=torch.int32)[1:]  # another alignment than the key's
        log(f"bits {bits} {nR} x {nS} shift {shift}")
        _native.tune_set("hash.bits", bits, local=True)
        try:
            pairs = J.hash_join(J.Relation(one), J.Relation(many, rid=rid))
        finally:
            _native.tune_set("hash.bits", None, local=True)
        row = torch.full((nS,), -1, dtype=torch.int64, device="cuda")
        row[pairs[:, 1].long() - 1] = pairs[:, 0].long()
        want = _lookup(one, many)
        assert pairs.shape[0] == int((want >= 0).sum()) and torch.equal(row, want)


@gpu
@pytest.mark.parametrize("jobs", [1, 70, 700])
def test_batch_of_packed_columns(jobs):
    """Joins at every alignment of the packed columns; 70 joins of up to 2^8 and 700 of up to 2^5
    partitions lie on both sides of one pass of the start computation."""
    from paper_1904_11201_amd import join as J
    need_gpu()
    g = torch.Generator()
    g.manual_seed(jobs)
    bits = 8 if jobs <= 70 else 5
    nR = torch.randint(1, 3000, (jobs,), generator=g).tolist()
    nS = torch.randint(0, 5000, (jobs,), generator=g).tolist()
    roffs, soffs, one, many = [0], [0], [], []
    for r, s in zip(nR, nS):
        roffs.append(roffs[-1] + r)
        soffs.append(soffs[-1] + s)
        one.append(torch.randperm(r, generator=g).to(torch.int32))
        many.append(torch.randint(-2, r + 2, (s,), generator=g).to(torch.int32))
    rk, sk = torch.cat(one).cuda(), torch.cat(many).cuda()
    rr = torch.arange(rk.numel(), device="cuda", dtype=torch.int32)
    sr = torch.arange(sk.numel(), device="cuda", dtype=torch.int32)
    log(f"batch of {jobs}")
    b = J.Batch.packed(rk, roffs, sk, soffs, bits=[bits] * jobs, rrids=rr, srids=sr)
    offs = b.count().tolist()
    pairs = torch.empty((offs[-1], 2), dtype=torch.int32, device="cuda")
    b.materialize(pairs)
    row = torch.full((sk.numel(),), -1, dtype=torch.int64)
    row[pairs[:, 1].cpu().long()] = pairs[:, 0].cpu().long()
    for j in range(jobs):
        want = _lookup(one[j], many[j])
        want = torch.where(want >= 0, want + roffs[j], want)
        assert torch.equal(row[soffs[j]:soffs[j + 1]], want), j
        assert offs[j + 1] - offs[j] == int((want >= 0).sum()), j
