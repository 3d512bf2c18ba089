"""Skewed columns of the region-pruned theta join: frequent values and most rows in a sliver of the
range, where buckets are made between quantiles of a sorted sample; against the oracle, and against
the time of uniform columns."""
import time

import numpy as np
import pytest
import torch

import oracle
from paper_1904_11201_amd import datagen
from tests.gpu_util import canon_gpu, dev_rel, gpu, log, need_gpu

TOP, LOW = (1 << 31) - 1, -(1 << 31)
SHAPES = ["half one value", "hot neighbours", "hot extremes", "few values", "power", "log-normal", "spike", "constant"]


def _column(shape, n, g):
    x = g.integers(0, 1 << 24, n)
    if shape == "half one value":
        x[::2] = 777_777
    elif shape == "hot neighbours":  # values beside each other, each of several buckets, and their gaps
        x[::3] = 5000
        x[1::3] = 5001 + 2 * g.integers(0, 3, len(x[1::3]))
    elif shape == "hot extremes":
        x[::4], x[1::4], x[2::4] = TOP, LOW, TOP - 1
    elif shape == "few values":
        x = g.integers(0, 37, n) * 100_003
    elif shape == "power":
        x = g.random(n) ** 16 * (1 << 30)
    elif shape == "log-normal":
        x = np.minimum(np.exp(g.normal(8, 3, n)), 2e9)
    elif shape == "spike":
        x = np.where(g.random(n) < 0.9, x % 3000, x * 100)
    elif shape == "constant":
        x[:] = -5
    return g.permutation(x).astype(np.int32)


def _sides(shape, nR, nS, seed=3):
    """R: half its rows from S's values and their neighbours; c among few values."""
    g = np.random.default_rng(seed)
    S = datagen.Rel(key=_column(shape, nS, g), key2=g.integers(0, 50, nS).astype(np.int32),
                    rid=g.permutation(nS).astype(np.int32))
    near = g.choice(S.key, nR - nR // 2).astype(np.int64) + g.integers(-1, 2, nR - nR // 2)
    rk = np.concatenate([_column(shape, nR // 2, g), np.clip(near, LOW, TOP)])
    R = datagen.Rel(key=g.permutation(rk).astype(np.int32), key2=g.integers(0, 50, nR).astype(np.int32),
                    rid=g.permutation(nR).astype(np.int32))
    return R, S


@gpu
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("nR,nS", [(200, 150_000), (9000, 4100), (61, 1 << 20)])
def test_skewed_columns(shape, nR, nS):
    need_gpu()
    from paper_1904_11201_amd import join as J
    R, S = _sides(shape, nR, nS)
    for A, B in ((R, S), (S, R)):
        dA, dB = dev_rel(A), dev_rel(B)
        for op_a, w, op_c in (("band", 2, "eq"), ("eq", 0, "eq"), ("lt", 0, "none"), ("ne", 0, "eq")):
            log(f"skew, {shape}: {A.n} x {B.n} {op_a}/{op_c}")
            pred = J.Pred(op_a, w, op_c)
            n, _ = oracle.theta_nlj(A.key, B.key, op_a, w=w, Rc=A.key2, Sc=B.key2, op_c=op_c, want_pairs=False)
            ws = J.workspace(J.JOIN_KIND_THETA_REGION, A.n, B.n, pred)
            assert J.join_count(J.JOIN_KIND_THETA_REGION, dA, dB, pred, ws) == n
            if n > 6_000_000:
                continue
            _, ref = oracle.theta_nlj(A.key, B.key, op_a, w=w, Rc=A.key2, Sc=B.key2, op_c=op_c, Rrid=A.rid, Srid=B.rid)
            assert np.array_equal(canon_gpu(J.theta_join(dA, dB, pred, region=True)), ref)


@gpu
@pytest.mark.parametrize("shape", ["half one value", "power"])
def test_a_skewed_column_does_not_dominate(shape):
    """1K x 1M: a skewed S takes at most 6 times a uniform one's time (one workgroup merging most of S
    took 140 and 85 times)."""
    need_gpu()
    from paper_1904_11201_amd import join as J
    pred = J.Pred("band", 0)
    R = dev_rel(datagen.small_random(5, 1000, 1, 0, 1 << 24)[0])
    took = {}
    for name in ("uniform", shape):
        S = dev_rel(datagen.Rel(key=_column(name, 1 << 20, np.random.default_rng(4))))
        ws = J.workspace(J.JOIN_KIND_THETA_REGION, R.n, S.n, pred)
        log(f"time of {name} S")
        runs = []
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            J.join_count(J.JOIN_KIND_THETA_REGION, R, S, pred, ws)
            runs.append(time.perf_counter() - t0)
        took[name] = min(runs)
    log(f"us: {[(k, round(v * 1e6)) for k, v in took.items()]}")
    assert took[shape] < 6 * took["uniform"]
