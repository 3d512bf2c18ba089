"""join_hash_noalloc at the edge of its static array: the partitioned join that comes closest to 64 MiB
from below with probe slices of 32K rows, whose smaller slices need 33 KB more."""
import torch

from tests.gpu_util import gpu, log, need_gpu


@gpu
def test_the_largest_joins_still_fit():
    need_gpu()
    from paper_1904_11201_amd import join as J
    nR, nS = 7_129_189, 1_175_889
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    R = J.Relation(torch.randperm(nR, device="cuda", generator=g).to(torch.int32))
    S = J.Relation(torch.randint(0, 2 * nR, (nS,), device="cuda", dtype=torch.int32, generator=g))
    n = int((S.key < nR).sum())
    out = torch.empty((n, 2), dtype=torch.int32, device="cuda")
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    log(f"noalloc {nR} x {nS}, {J.join_workspace_bytes(J.JOIN_KIND_HASH, nR, nS)} bytes")
    J.join_hash_noalloc(R, S, out, count)
    assert int(count[0]) == n
    assert torch.equal(R.key[out[:, 0].long()], S.key[out[:, 1].long()])
    assert out[:, 1].unique().numel() == n
