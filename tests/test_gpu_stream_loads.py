"""Joins on both sides of the size from which the probe tuples are read non-temporally (320 MiB of
tuples), in the plain, resident, pre-filtered and batched passes, against a lookup in torch."""
import pytest
import torch

from tests.gpu_util import gpu, log, need_gpu

LINE = (320 << 20) // 8


@gpu
@pytest.mark.parametrize("extra", [0, 1])
@pytest.mark.parametrize("how", ["plain", "resident", "prefilter", "batch"])
def test_both_sides_of_the_streaming_size(extra, how):
    from paper_1904_11201_amd import join as J
    need_gpu()
    g = torch.Generator(device="cuda")
    g.manual_seed(extra + 2)
    nR = 1_000_003
    nS = LINE - nR + extra
    hit = 0.01 if how == "prefilter" else 1.0
    one = torch.randperm(nR, device="cuda", generator=g).to(torch.int32)
    many = torch.randint(0, int(nR / hit), (nS,), device="cuda", dtype=torch.int32, generator=g)
    log(f"{how} {nR} x {nS}")
    R, S = J.Relation(one), J.Relation(many)
    if how == "plain":
        pairs = J.hash_join(R, S)
    elif how == "prefilter":
        pairs = J.hash_join(R, S, prefilter=True)
    elif how == "resident":
        pairs = J.ResidentBuild(R).probe(S)
    else:
        pairs = J.hash_join_batch([J.Job(R, S)])[0]
    at = torch.empty(nR, device="cuda", dtype=torch.int64)
    at[one.long()] = torch.arange(nR, device="cuda")
    want = torch.where(many < nR, at[many.long().clamp_(max=nR - 1)], -1)
    row = torch.full((nS,), -1, dtype=torch.int64, device="cuda")
    row[pairs[:, 1].long()] = pairs[:, 0].long()
    assert pairs.shape[0] == int((want >= 0).sum()) and torch.equal(row, want)
