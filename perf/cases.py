"""The work this library is measured on: joins as programs call them, from the smallest to the
largest, each through a public entry point of paper_1904_11201_amd.join.

The order of a join's pairs is left open by the library, so a program that keeps a result first
gives it a form of its own.  Here that form is

* for a many-to-one join (every row of one side matches at most one row of the other: a foreign
  key looked up), the row id found for each row of the "many" side, -1 for none;
* for a band join, the pairs in ascending order, in a buffer of a fixed size the program keeps;
* for a count or a batch's sizes, the numbers themselves.

Keys, row ids and sizes follow paper_1904_11201_amd.datagen (uniform keys, permutations, bounded
Zipf ranks, log-uniform batch sizes) and are made on the device from the seed alone.

Kinds of case
  equi       hash_join, many-to-one: unique keys on one side ("many" names the other)
  count      join_count of the hash join (SELECT COUNT(*), or sizing a result)
  resident   ResidentBuild.probe of a build kept partitioned
  batch      Batch.packed: count pass, exact allocation, write pass of many joins at once
  band       theta_join on |R.a - S.a| <= w [and R.c < S.c], nested loop or region-pruned
  theta      join_count of a theta join
"""
import math

import torch

from paper_1904_11201_amd import join as J

M = 1 << 20
DOMAIN = 1 << 24  # theta columns are uniform in [0, DOMAIN)


def listed():
    return [
        # the smallest requests of the serving stream: launches and host time
        {"name": "equi_1k", "kind": "equi", "nR": 1000, "nS": 4000, "many": "S", "zipf": False,
         "rids": False, "match": 1.0, "prefilter": False},
        # the plain single request, 64K x 64K; the build side repeats its keys
        {"name": "equi_64k", "kind": "equi", "nR": 65536, "nS": 65536, "many": "R", "zipf": False,
         "rids": True, "match": 1.0, "prefilter": False},
        # a star join: a dimension table of 100,000 rows against a fact table
        {"name": "star_100k_16m", "kind": "equi", "nR": 100_000, "nS": 16 * M, "many": "S",
         "zipf": False, "rids": False, "match": 1.0, "prefilter": False},
        # an ordinary join, sizes not a multiple of anything, with row id columns
        {"name": "equi_1m_4m", "kind": "equi", "nR": 1_000_003, "nS": 4_000_037, "many": "S",
         "zipf": False, "rids": True, "match": 0.9, "prefilter": False},
        # a large join with hot keys, half the size of the 16M x 64M benchmark
        {"name": "equi_8m_32m_zipf", "kind": "equi", "nR": 8 * M, "nS": 32 * M, "many": "S",
         "zipf": True, "rids": False, "match": 1.0, "prefilter": False},
        # the 16M x 64M benchmark join, its exact size
        {"name": "count_16m_64m", "kind": "count", "nR": 16 * M, "nS": 64 * M, "zipf": False,
         "match": 0.9},
        # the pre-filter's workload: 1% of the probe rows match
        {"name": "prefilter_1m_64m", "kind": "equi", "nR": M, "nS": 64 * M, "many": "S",
         "zipf": False, "rids": False, "match": 0.01, "prefilter": True},
        # serving: a request against a build that stays resident
        {"name": "resident_1m_64k", "kind": "resident", "nR": M, "nS": 65536},
        # many independent joins in one set of launches, sizes log-uniform
        {"name": "batch_256", "kind": "batch", "jobs": 256, "lo": 1024, "hi": M},
        # band joins, region-pruned: the 1M x 1M benchmark, and the size of a large result
        {"name": "band_1m", "kind": "band", "nR": M, "nS": M, "w": 8, "c": True, "region": True},
        {"name": "band_count_4m", "kind": "theta", "nR": 4 * M, "nS": 4 * M, "op": "band", "w": 8,
         "c": False, "region": True},
        # the nested loop, the default of theta_join, at its ordinary size
        {"name": "band_nested_100k", "kind": "band", "nR": 100_000, "nS": 100_000, "w": 8, "c": True,
         "region": False},
    ]


def _size(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))


def draw(rng):
    kind = rng.choice(["equi", "equi", "equi", "count", "resident", "batch", "band", "band", "theta"])
    if kind == "equi":
        prefilter = rng.random() < 0.15
        nR = _size(rng, 1000, 2 * M if prefilter else 8 * M)
        nS = _size(rng, 1000, 16 * M)
        many = "S" if prefilter else rng.choice(["S", "S", "R"])
        return {"kind": kind, "nR": nR, "nS": nS, "many": many, "zipf": rng.random() < 0.25,
                "rids": rng.random() < 0.5, "match": rng.choice([1.0, 1.0, 0.5, 0.01]),
                "prefilter": prefilter}
    if kind == "count":
        return {"kind": kind, "nR": _size(rng, 1000, 16 * M), "nS": _size(rng, 1000, 64 * M),
                "zipf": rng.random() < 0.25, "match": rng.choice([0.9, 0.9, 0.5])}
    if kind == "resident":
        return {"kind": kind, "nR": _size(rng, 200_000, 8 * M), "nS": _size(rng, 1000, 8 * M)}
    if kind == "batch":
        return {"kind": kind, "jobs": rng.randrange(8, 257), "lo": 1024, "hi": _size(rng, 16384, M)}
    if kind == "band":
        region = rng.random() < 0.7
        hi = M if region else 100_000
        return {"kind": kind, "nR": _size(rng, 1000, hi), "nS": _size(rng, 1000, hi),
                "w": rng.choice([0, 1, 8, 8, 100]), "c": rng.random() < 0.5, "region": region}
    region = rng.random() < 0.7
    op = rng.choice(["band", "lt", "ge"])
    hi = 4 * M if region and op == "band" else 100_000
    return {"kind": "theta", "nR": _size(rng, 1000, hi), "nS": _size(rng, 1000, hi), "op": op, "w": 8,
            "c": rng.random() < 0.3, "region": region}


# ------------------------------------------------------------------------------------ inputs --
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _uniform(g, n, hi):
    return torch.randint(0, hi, (n,), device="cuda", dtype=torch.int32, generator=g)


def _perm(g, n):
    return torch.randperm(n, device="cuda", generator=g).to(torch.int32)


def _pick(g, n, domain, zipf):
    """n positions in [0, domain): uniform, or bounded Zipf(1.0) ranks by inverse CDF."""
    if not zipf:
        return torch.randint(0, domain, (n,), device="cuda", generator=g)
    harm = torch.cumsum(1.0 / torch.arange(1, domain + 1, device="cuda", dtype=torch.float64), 0)
    u = torch.rand(n, device="cuda", dtype=torch.float64, generator=g) * harm[-1]
    return torch.searchsorted(harm, u, right=True).clamp_(max=domain - 1)


def _many_to_one(g, n_one, n_many, zipf, match):
    """Unique keys of the "one" side, and keys of the "many" side of which about `match` occur
    among them.  The unique keys are spread over a domain 1 / match times their number."""
    step = max(1, round(1 / match))
    one = _perm(g, n_one) * step
    if match == 1.0 or zipf:
        many = one[_pick(g, n_many, n_one, zipf)]
        if match < 1.0:
            miss = torch.rand(n_many, device="cuda", generator=g) >= match
            many = torch.where(miss, -1 - many, many)
    elif step > 1:
        many = _uniform(g, n_many, n_one * step)
    else:
        many = _uniform(g, n_many, round(n_one / match))
    return one, many


def _theta_side(g, n, c):
    return J.Relation(_uniform(g, n, DOMAIN), _uniform(g, n, DOMAIN) if c else None)


def _pred(case):
    return J.Pred(case.get("op", "band"), case["w"], "lt" if case["c"] else "none")


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "equi":
        n_many, n_one = (case["nR"], case["nS"]) if case["many"] == "R" else (case["nS"], case["nR"])
        one, many = _many_to_one(g, n_one, n_many, case["zipf"], case["match"])
        rk, sk = (many, one) if case["many"] == "R" else (one, many)
        rr = _perm(g, case["nR"]) if case["rids"] else None
        sr = _perm(g, case["nS"]) if case["rids"] else None
        return {"case": case, "R": J.Relation(rk, rid=rr), "S": J.Relation(sk, rid=sr)}
    if kind == "count":
        one, many = _many_to_one(g, case["nR"], case["nS"], case["zipf"], case["match"])
        ws = J.workspace(J.JOIN_KIND_HASH, case["nR"], case["nS"])
        return {"case": case, "R": J.Relation(one), "S": J.Relation(many), "ws": ws}
    if kind == "resident":
        one, many = _many_to_one(g, case["nR"], case["nS"], False, 1.0)
        return {"case": case, "R": J.Relation(one), "build": J.ResidentBuild(J.Relation(one)),
                "S": J.Relation(many)}
    if kind == "batch":
        return _prepare_batch(case, g)
    R, S = _theta_side(g, case["nR"], case["c"]), _theta_side(g, case["nS"], case["c"])
    state = {"case": case, "R": R, "S": S, "pred": _pred(case)}
    if kind == "theta":
        state["kind"] = J.JOIN_KIND_THETA_REGION if case["region"] else J.JOIN_KIND_THETA
        state["ws"] = J.workspace(state["kind"], case["nR"], case["nS"], state["pred"])
    else:
        state["kept"] = torch.empty(_kept(case), dtype=torch.int64, device="cuda")
    return state


def _kept(case):
    """Pairs a band join's buffer holds: the average and some room."""
    return int(1.2 * _expected_pairs(case)) + 1000


def _batch_sizes(case):
    """Sizes of the batch's joins: log-uniform, the same for every seed (they set the work)."""
    g = torch.Generator()
    g.manual_seed(case["jobs"] * 7919 + case["hi"])
    u = torch.rand(2, case["jobs"], generator=g, dtype=torch.float64)
    n = torch.exp(math.log(case["lo"]) + u * math.log(case["hi"] / case["lo"])).long()
    return n[0].tolist(), n[1].tolist()


def _prepare_batch(case, g):
    nR, nS = _batch_sizes(case)
    ones, manys, roffs, soffs = [], [], [0], [0]
    for j, (r, s) in enumerate(zip(nR, nS)):
        one, many = _many_to_one(g, r, s, j % 10 == 9, 1.0)
        ones.append(one)
        manys.append(many)
        roffs.append(roffs[-1] + r)
        soffs.append(soffs[-1] + s)
    rk, sk = torch.cat(ones), torch.cat(manys)
    rr = torch.arange(rk.numel(), device="cuda", dtype=torch.int32)  # row ids in the packed columns
    sr = torch.arange(sk.numel(), device="cuda", dtype=torch.int32)
    return {"case": case, "rk": rk, "sk": sk, "roffs": roffs, "soffs": soffs,
            "batch": J.Batch.packed(rk, roffs, sk, soffs, rrids=rr, srids=sr)}


# --------------------------------------------------------------------------------- the passes --
def _lookup(pairs, n, many):
    """The row id found for each of the n rows of the "many" side (column `many` of the pairs)."""
    row = torch.full((n,), -1, dtype=torch.int32, device=pairs.device)
    return row.scatter_(0, pairs[:, many], pairs[:, 1 - many])


def _in_order(pairs, kept):
    """The pairs in ascending (S row, R row) order, one 64-bit key a pair, then -1."""
    n = pairs.shape[0]
    kept[:n] = pairs.view(torch.int64).reshape(-1).sort().values
    kept[n:] = -1
    return {"pairs": n, "kept": kept}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "equi":
        pairs = J.hash_join(state["R"], state["S"], prefilter=case["prefilter"])
        n, many = (case["nR"], 0) if case["many"] == "R" else (case["nS"], 1)
        return {"pairs": pairs.shape[0], "row": _lookup(pairs, n, many)}
    if kind == "count":
        return {"pairs": J.join_count(J.JOIN_KIND_HASH, state["R"], state["S"], None, state["ws"])}
    if kind == "resident":
        pairs = state["build"].probe(state["S"])
        return {"pairs": pairs.shape[0], "row": _lookup(pairs, case["nS"], 1)}
    if kind == "batch":
        batch = state["batch"]
        offsets = batch.count()
        pairs = torch.empty((int(offsets[-1]), 2), dtype=torch.int32, device="cuda")
        batch.materialize(pairs)
        return {"offsets": offsets, "row": _lookup(pairs, state["sk"].numel(), 1)}
    if kind == "band":
        return _in_order(J.theta_join(state["R"], state["S"], state["pred"], region=case["region"]),
                         state["kept"])
    return {"pairs": J.join_count(state["kind"], state["R"], state["S"], state["pred"], state["ws"])}


def _expected_pairs(case):
    """Pairs of a case, on average over the seeds."""
    if case["kind"] == "equi":
        return (case["nR"] if case["many"] == "R" else case["nS"]) * case["match"]
    if case["kind"] == "resident":
        return case["nS"]
    if case["kind"] == "batch":
        return sum(_batch_sizes(case)[1])
    if case["kind"] == "band":
        return case["nR"] * case["nS"] * (2 * case["w"] + 1) / DOMAIN * (0.5 if case["c"] else 1.0)
    return 0  # a count returns one number


def work(case):
    """Columns read once, pairs (8 bytes) written once, and what the program makes of them: the
    lookup column or the ordered pairs written once."""
    out = _expected_pairs(case)
    if case["kind"] == "batch":
        nR, nS = _batch_sizes(case)
        return {"bytes": 8 * (sum(nR) + sum(nS)) + 8 * out + 4 * sum(nS), "flops": 0}
    rows = case["nR"] + case["nS"]
    if case["kind"] == "equi":
        kept = case["nR"] if case["many"] == "R" else case["nS"]
        return {"bytes": (8 if case["rids"] else 4) * rows + 8 * out + 4 * kept, "flops": 0}
    if case["kind"] == "resident":
        return {"bytes": 8 * case["nR"] + 4 * case["nS"] + 12 * out, "flops": 0}
    if case["kind"] == "count":
        return {"bytes": 4 * rows, "flops": 0}
    return {"bytes": (8 if case["c"] else 4) * rows + 16 * out, "flops": 0}


# ---------------------------------------------------------------------------------- in torch --
def _find(one, one_rid, many):
    """Row id of each "many" key among the unique keys, -1 for none."""
    keys, order = one.long().sort()
    at = torch.searchsorted(keys, many.long()).clamp_(max=keys.numel() - 1)
    rid = order if one_rid is None else one_rid.long()[order]
    return torch.where(keys[at] == many.long(), rid[at], torch.full_like(at, -1))


def _window(R, S, pred):
    """First and last + 1 position, in S sorted by a, of the rows with op_a(R.a, S.a)."""
    keys, order = S.key.long().sort()
    a = R.key.long()
    zero, end = torch.zeros_like(a), torch.full_like(a, keys.numel())
    if pred.op_a == "band":
        return torch.searchsorted(keys, a - pred.w), torch.searchsorted(keys, a + pred.w, right=True), order
    if pred.op_a == "lt":
        return torch.searchsorted(keys, a, right=True), end, order
    return zero, torch.searchsorted(keys, a, right=True), order  # ge


def _theta_exact(state, count_only):
    R, S, pred = state["R"], state["S"], state["pred"]
    lo, hi, order = _window(R, S, pred)
    if pred.op_c == "none" and count_only:
        return {"pairs": int((hi - lo).sum())}
    total, out, step = 0, [], max(1, int(1e8 // max(1, int((hi - lo).max()))))
    for b in range(0, R.n, step):
        n = (hi - lo)[b:b + step]
        r = torch.repeat_interleave(torch.arange(b, b + n.numel(), device="cuda"), n)
        first = torch.repeat_interleave(lo[b:b + step] - (n.cumsum(0) - n), n)
        s = order[first + torch.arange(r.numel(), device="cuda")]
        if pred.op_c != "none":
            keep = R.key2[r] < S.key2[s]
            r, s = r[keep], s[keep]
        total += r.numel()
        if not count_only:
            out.append((s << 32) | r)
    if count_only:
        return {"pairs": total}
    state["kept"].fill_(-1)
    state["kept"][:total] = torch.cat(out).sort().values
    return {"pairs": total, "kept": state["kept"]}


def exact(case, seed):
    state = prepare(case, seed)
    kind = case["kind"]
    if kind in ("band", "theta"):
        return _theta_exact(state, kind == "theta")
    if kind == "batch":
        rows, sizes = [], [0]
        ro, so = state["roffs"], state["soffs"]
        for j in range(case["jobs"]):
            row = _find(state["rk"][ro[j]:ro[j + 1]], None, state["sk"][so[j]:so[j + 1]])
            sizes.append(sizes[-1] + int((row >= 0).sum()))
            rows.append(torch.where(row >= 0, row + ro[j], row))
        return {"offsets": torch.tensor(sizes, device="cuda"), "row": torch.cat(rows).to(torch.int32)}
    if kind == "equi" and case["many"] == "R":
        one, many = state["S"], state["R"]
    else:
        one, many = state["R"], state["S"]
    row = _find(one.key, one.rid, many.key).to(torch.int32)
    pairs = int((row >= 0).sum())
    if kind == "count":
        return {"pairs": pairs}
    if many.rid is not None:
        row = torch.empty_like(row).scatter_(0, many.rid.long(), row)
    return {"pairs": pairs, "row": row}
