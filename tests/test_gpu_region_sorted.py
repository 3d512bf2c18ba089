"""The sorted form of the region-pruned theta join at the edges of its cases, against the oracle:
one LDS sort and partitioned sides, buckets larger than one sort (merged), outliers beyond the
sampled range, intervals walked lane by lane and by the whole wave, with and without column c."""
import numpy as np
import pytest

import oracle
from paper_1904_11201_amd import datagen
from tests.gpu_util import canon_gpu, dev_rel, gpu, log, need_gpu

CAP = 4096   # rows of one LDS sort
SERIAL = 32  # longest interval walked lane by lane


def _check(R, S, op_a, w, op_c, what):
    from paper_1904_11201_amd.join import Pred, theta_join
    log(f"region {what} {op_a}/{op_c} w={w}")
    n, ref = oracle.theta_nlj(R.key, S.key, op_a, w=w, Rc=R.key2, Sc=S.key2, op_c=op_c, Rrid=R.rid,
                              Srid=S.rid)
    got = canon_gpu(theta_join(dev_rel(R), dev_rel(S), Pred(op_a, w, op_c), region=True))
    assert len(got) == n and np.array_equal(got, ref)


@gpu
@pytest.mark.parametrize("nR,nS", [(CAP, CAP), (CAP + 1, 3), (3, CAP + 1), (CAP + 1, CAP + 1), (9001, 5003)])
@pytest.mark.parametrize("op_a,op_c", [("band", "lt"), ("band", "none"), ("eq", "none"), ("ge", "none"),
                                       ("lt", "ge"), ("ne", "eq")])
def test_sizes_around_one_sort(nR, nS, op_a, op_c):
    need_gpu()
    R, S = datagen.small_random(nR + 7 * nS, nR, nS, -20000, 20000, with_c=True, rid_mode="random")
    _check(R, S, op_a, 3 if op_a == "band" else 0, op_c, f"{nR} x {nS}")


@gpu
@pytest.mark.parametrize("shape", ["one value", "dense under an outlier", "hot value", "two outliers"])
def test_buckets_larger_than_one_sort(shape):
    """Buckets of several chunks: the last chunk's workgroup merges them (2, 3 and 5 chunks)."""
    need_gpu()
    R, S = datagen.small_random(5, 700, 20000, 0, 3000, with_c=True, rid_mode="random")
    if shape == "one value":
        S.key[:] = 1500
    elif shape == "dense under an outlier":
        S.key[:] %= 40
        S.key[0] = (1 << 31) - 1
        S.key[7] = -(1 << 31)
    elif shape == "hot value":
        S.key[3000:12500] = 777
    else:
        S.key[5] = (1 << 31) - 1
        R.key[6] = -(1 << 31)
    for sides in ((R, S), (S, R)):
        _every_operator(*sides, shape)


def _every_operator(R, S, shape):
    for op_a, w, op_c in (("band", 2, "lt"), ("le", 0, "none"), ("eq", 0, "none"), ("ne", 0, "gt")):
        _check(R, S, op_a, w, op_c, shape)


@gpu
@pytest.mark.parametrize("hot", [63, 64, 65, 3000])
@pytest.mark.parametrize("nS", [65, 4095, 4096])
def test_crowded_bins(hot, nS):
    """A frequent value among widely spread ones: ranked inside its bin up to 64 rows, by the
    bitonic network beyond."""
    need_gpu()
    R, S = datagen.small_random(hot + nS, 900, nS, -(1 << 31), (1 << 31) - 1, with_c=True, rid_mode="random")
    S.key[:min(hot, nS)] = 12345
    S.key[nS // 2:] = np.random.default_rng(hot).permutation(S.key[nS // 2:])
    R.key[:40] = 12345
    R.key[40:80] = S.key[-40:]
    _every_operator(R, S, f"hot {hot} of {nS}")


@gpu
@pytest.mark.parametrize("length", [SERIAL - 1, SERIAL, SERIAL + 1, 700])
@pytest.mark.parametrize("op_c", ["none", "lt"])
def test_interval_lengths(length, op_c):
    """S holds every value once, so a band of w reaches 2w + 1 rows (fewer at the ends)."""
    need_gpu()
    R, S = datagen.small_random(length, 1500, 6000, 0, 6000, with_c=True, rid_mode="random")
    S.key[:] = np.random.default_rng(length).permutation(6000).astype(np.int32)
    _check(R, S, "band", length // 2, op_c, f"length {length}")
