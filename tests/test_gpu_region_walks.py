"""Long intervals of the region-pruned theta join under a condition on column c: walked by R rows
where R is sparse, by S rows where the intervals overlap, shared by several units where R is small;
against the oracle, and against the time of the same join without the condition."""
import time

import numpy as np
import pytest
import torch

import oracle
from paper_1904_11201_amd import datagen
from tests.gpu_util import canon_gpu, dev_rel, gpu, log, need_gpu


def _check(R, S, op_a, w, op_c, what):
    from paper_1904_11201_amd import join as J
    log(f"region walk, {what}: {R.n} x {S.n} {op_a}/{op_c} w={w}")
    n, ref = oracle.theta_nlj(R.key, S.key, op_a, w=w, Rc=R.key2, Sc=S.key2, op_c=op_c, Rrid=R.rid, Srid=S.rid)
    pred, dR, dS = J.Pred(op_a, w, op_c), dev_rel(R), dev_rel(S)
    ws = J.workspace(J.JOIN_KIND_THETA_REGION, R.n, S.n, pred)
    assert J.join_count(J.JOIN_KIND_THETA_REGION, dR, dS, pred, ws) == n
    got = canon_gpu(J.theta_join(dR, dS, pred, region=True))
    assert np.array_equal(got, ref)


@gpu
@pytest.mark.parametrize("nR", [1, 3, 63, 65, 300, 1025])
@pytest.mark.parametrize("op_c", ["lt", "ge", "eq"])
def test_sparse_r(nR, op_c):
    """Intervals of about 120 rows, hundreds of rows apart (by R rows), with R blocks cut into up to
    64 shares; the widest band reaches all of S (by S rows)."""
    need_gpu()
    R, S = datagen.small_random(nR, nR, 60_000, 0, 1 << 20, with_c=True, rid_mode="random")
    S.key2[:] %= 5000
    R.key2[:] %= 5000
    for w in (8, 1000, 1 << 20) if op_c == "eq" else (8, 1000):
        _check(R, S, "band", w, op_c, "sparse R")


@gpu
@pytest.mark.parametrize("nR,nS,w", [(500, 500, 64), (2000, 6000, 3000), (6000, 2000, 200), (70_000, 3000, 100)])
def test_overlapping_intervals(nR, nS, w):
    """By S rows: whole batches of 64 rows inside every interval of the wave, and their ends."""
    need_gpu()
    R, S = datagen.small_random(nR + nS, nR, nS, 0, 20_000, with_c=True, rid_mode="random")
    S.key2[:] %= 100
    R.key2[:] %= 100
    _check(R, S, "band", w, "eq", "overlapping")


@gpu
@pytest.mark.parametrize("op_a", ["eq", "ne", "lt", "ge", "band"])
def test_frequent_values_among_others(op_a):
    """Intervals of 0, 1 and thousands of rows in one wave."""
    need_gpu()
    R, S = datagen.small_random(17, 400, 9000, 0, 4000, with_c=True, rid_mode="random")
    S.key2[:] %= 1000
    R.key2[:] %= 1000
    S.key[1000:6000] = 2000
    S.key[6000:6100] = 2001
    R.key[::3] = 2000
    _check(R, S, op_a, 1 if op_a == "band" else 0, "eq", "frequent values")


@gpu
@pytest.mark.parametrize("w", [1000, 100_000])
def test_a_condition_on_c_does_not_dominate_a_sparse_r(w):
    """1K x 1M: with c at most 8 times the time without (walking the gaps between the intervals took
    47 and 93 times)."""
    need_gpu()
    from paper_1904_11201_amd import join as J
    R, S = (dev_rel(datagen.small_random(5, n, 1, 0, 1 << 24, with_c=True)[0]) for n in (1000, 1 << 20))
    took = {}
    for op_c in ("none", "lt"):
        pred = J.Pred("band", w, op_c)
        ws = J.workspace(J.JOIN_KIND_THETA_REGION, R.n, S.n, pred)
        log(f"sparse R, w={w}, op_c {op_c}")
        runs = []
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            J.join_count(J.JOIN_KIND_THETA_REGION, R, S, pred, ws)
            runs.append(time.perf_counter() - t0)
        took[op_c] = min(runs)
    log(f"without c {took['none'] * 1e6:.0f} us, with c {took['lt'] * 1e6:.0f} us")
    assert took["lt"] < 8 * took["none"]
