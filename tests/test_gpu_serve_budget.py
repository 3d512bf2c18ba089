"""A serving budget that holds a join of a small build unpartitioned, but not its partitioned tuples."""
import pytest
import torch

from tests.gpu_util import gpu, log, need_gpu


@gpu
@pytest.mark.parametrize("resident", [False, True])
def test_a_small_build_fits_the_budget_it_always_fitted(resident):
    need_gpu()
    from paper_1904_11201_amd import _native
    from paper_1904_11201_amd import join as J
    from paper_1904_11201_amd.serve import BudgetError, Engine, Request
    nR, nS = 100_000, 4_000_000
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    R = J.Relation(torch.randperm(nR, device="cuda", generator=g).to(torch.int32))
    S = J.Relation(torch.randint(0, 100 * nR, (nS,), device="cuda", dtype=torch.int32, generator=g))
    n = int((S.key < nR).sum())
    assert J.join_workspace_bytes(J.JOIN_KIND_HASH, nR, nS) > 8 * nS
    req = Request(0, "hash", S, None if resident else R, 0 if resident else -1)
    budget = (1 << 20) + 8 * n
    log(f"serving {nR} x {nS} within {budget} bytes")
    engine = Engine([R], slots=2, budget_bytes=budget)
    (res,), _ = engine.serve([req], open_loop=False)
    assert res.count == n and engine.peak <= budget and engine.reserved == 0
    assert torch.equal(R.key[res.pairs[:, 0].long()], S.key[res.pairs[:, 1].long()])
    assert res.pairs[:, 1].unique().numel() == n
    with pytest.raises(BudgetError):
        Engine([R], budget_bytes=8 * n).serve([req], open_loop=False)
    assert _native.tune_get("hash.single_max_chunks", -1) == -1
