"""Performance cases of the self-join: the calls that a program makes on new points.

A program hands the library points and a search distance, and each pass here does all that follows from it: the
grid is built and the result is taken (a handle keeps its counts, so a second count on one handle would measure
nothing). What stays outside is the points themselves, the choice of the distance, and the buffer that the pairs go
to, which a program with a result larger than it wants to hold keeps and passes again. The buffer has room for more
pairs than `s` neighbours a point give, and -1 past the last one.

Sizes: the benchmark's sets (uniform and exponential at 2M points in 2 to 4 dimensions, the 10M-point exponential
set, the Gaussian mixtures at 1M points in 16 to 64 dimensions, 256 mixed problems in one batch, the index-free
mode in 16 dimensions), the small parity set (20,000 points), and the smallest call of the allocation-free entry
point. Points are drawn on the GPU by the recipes of workloads/generators.py. The distance is the one that gives
about `s` neighbours a point, the way a user tunes it: from the distances of some points to a part of the set.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2209_11287_amd import (selfjoin_batch_build, selfjoin_batch_count, selfjoin_batch_free,
                                  selfjoin_batch_pairs, selfjoin_build_grid, selfjoin_core_points, selfjoin_count,
                                  selfjoin_count_noalloc, selfjoin_free_grid, selfjoin_knn, selfjoin_pairs)

BATCH_DIMS = (2, 3, 4, 8, 16)


def listed():
    return [
        # The smallest call: a serving loop that must not allocate asks for the neighbour counts of a few points.
        {"name": "noalloc_uniform_d3_n1500", "kind": "noalloc", "dist": "uniform", "n": 1500, "d": 3, "s": 16.0,
         "path": "fp64_mfma"},
        # A small data set joined once: launches and host waits count as much as kernels.
        {"name": "join_uniform_d2_n20000", "kind": "join", "dist": "uniform", "n": 20000, "d": 2, "s": 29.0,
         "path": "fp64_mfma", "d2": False},
        # The benchmark's low-dimensional sets: evenly spread points, the whole pair list.
        {"name": "join_uniform_d2_n2M", "kind": "join", "dist": "uniform", "n": 2000000, "d": 2, "s": 64.0,
         "path": "fp64_mfma", "d2": False},
        # Skewed points, an odd number of them, with the distances that a weighted graph or a kernel sum needs.
        {"name": "join_expo_d4_n1999993_d2", "kind": "join", "dist": "expo", "n": 1999993, "d": 4, "s": 64.0,
         "path": "fp64_mfma", "d2": True},
        # The first half of density-based clustering: core flags only, with the count-only option set.
        {"name": "core_uniform_d3_n2000003", "kind": "core", "dist": "uniform", "n": 2000003, "d": 3, "s": 64.0,
         "path": "fp64_mfma", "min_pts": 60},
        # The largest set and result: 10M skewed points, about 10^9 pairs.
        {"name": "join_expo_d3_n10M", "kind": "join", "dist": "expo", "n": 10000000, "d": 3, "s": 100.0,
         "path": "fp64_mfma", "d2": False},
        # Clustered feature vectors: fewer dimensions indexed than there are, in FP64 and on the two
        # low-precision paths that a user takes for speed at high d (the result is the same set).
        {"name": "join_gmm_d16_n1M", "kind": "join", "dist": "gmm", "n": 1000000, "d": 16, "s": 50.0,
         "path": "fp64_mfma", "d2": False},
        {"name": "join_gmm_d32_n1M_fp32", "kind": "join", "dist": "gmm", "n": 1000000, "d": 32, "s": 50.0,
         "path": "fp32_mfma", "d2": False},
        {"name": "join_gmm_d64_n1M_bf16x3", "kind": "join", "dist": "gmm", "n": 1000000, "d": 64, "s": 50.0,
         "path": "bf16x3_mfma", "d2": False},
        # Neighbour lists with distances for a graph or a local density estimate.
        {"name": "knn_uniform_d3_n500009_k10", "kind": "knn", "dist": "uniform", "n": 500009, "d": 3, "s": 32.0,
         "path": "fp64_mfma", "k": 10},
        # The index-free mode: every ordered pair is a candidate, per-point counts.
        {"name": "count_noindex_expo_d16_n65536", "kind": "count", "dist": "expo", "n": 65536, "d": 16, "s": 32.0,
         "path": "fp64_mfma", "index_dims": -1},
        # Many independent problems of uneven size and dimension in one call.
        {"name": "batch_256_problems", "kind": "batch", "problems": 256, "mix": 0, "n_lo": 1000, "n_hi": 200000,
         "s": 32.0, "path": "fp64_mfma"},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["join", "join", "join", "join", "count", "count", "core", "knn", "noalloc", "noindex", "batch"])
    s = round(math.exp(rng.uniform(math.log(8.0), math.log(100.0))), 2)
    if kind == "batch":
        return {"kind": "batch", "problems": _log_uniform(rng, 8, 200), "mix": rng.randrange(1 << 20),
                "n_lo": 1000, "n_hi": _log_uniform(rng, 4000, 100000), "s": min(s, 32.0), "path": "fp64_mfma"}
    if kind == "noalloc":
        return {"kind": "noalloc", "dist": rng.choice(["uniform", "expo"]), "n": _log_uniform(rng, 500, 200000),
                "d": rng.randint(2, 4), "s": s, "path": "fp64_mfma"}
    if kind == "noindex":
        return {"kind": "count", "dist": "expo", "n": _log_uniform(rng, 1 << 11, 1 << 16), "d": rng.randint(8, 24),
                "s": s, "path": "fp64_mfma", "index_dims": -1}
    if kind == "knn":
        return {"kind": "knn", "dist": rng.choice(["uniform", "expo"]), "n": _log_uniform(rng, 2000, 1000000),
                "d": rng.randint(2, 4), "s": max(s, 16.0), "path": "fp64_mfma", "k": rng.randint(1, 32)}
    if kind == "core":
        return {"kind": "core", "dist": rng.choice(["uniform", "expo"]), "n": _log_uniform(rng, 1000, 4000000),
                "d": rng.randint(2, 4), "s": s, "path": "fp64_mfma", "min_pts": max(2, int(s * rng.uniform(0.5, 1.2)))}
    if rng.random() < 0.5:
        n, d, dist = _log_uniform(rng, 1000, 4000000), rng.randint(2, 5), rng.choice(["uniform", "expo"])
        path = rng.choice(["fp64_mfma", "fp64_mfma", "fp64_valu"])
    else:
        n, d, dist = _log_uniform(rng, 5000, 1000000), _log_uniform(rng, 6, 64), "gmm"
        path = rng.choice(["fp64_mfma", "fp64_mfma", "fp32_mfma", "bf16x3_mfma"])
    if kind == "count":
        return {"kind": "count", "dist": dist, "n": n, "d": d, "s": s, "path": path, "index_dims": 0}
    return {"kind": "join", "dist": dist, "n": n, "d": d, "s": s, "path": path, "d2": rng.random() < 0.3}


def _points(dist, n, d, gen):
    """n x d points on the GPU by the recipes of workloads/generators.py."""
    if dist == "gmm":
        centres = torch.rand((100, d), generator=gen, dtype=torch.float64, device="cuda")
        labels = torch.randint(0, 100, (n,), generator=gen, device="cuda")
        return centres[labels] + 0.02 * torch.randn((n, d), generator=gen, dtype=torch.float64, device="cuda")
    u = torch.rand((n, d), generator=gen, dtype=torch.float64, device="cuda")
    if dist == "expo":
        u = (torch.log1p(-u) / -40.0).clamp_(max=1.0)
    return u


def _distance(points, s):
    """The search distance for about `s` neighbours a point: a quantile of the distances from the first points to
    the first part of the set (the points come in no order)."""
    n, d = points.shape
    q, m = min(n, 1024), min(n, 65536)
    d2 = torch.zeros((q, m), dtype=torch.float64, device=points.device)
    for t in range(d):
        d2.add_((points[:q, t, None] - points[None, :m, t]).square_())
    pos = max(q + 1, int(round(q * (1.0 + s * m / n))))
    kth = torch.topk(d2.view(-1), min(pos, q * m), largest=False, sorted=False).values.max()
    return math.sqrt(float(kth))


def _mix(case):
    """Sizes and dimensions of a batch's problems: n log-uniform, d from BATCH_DIMS."""
    rng = random.Random(case["mix"])
    return [(_log_uniform(rng, case["n_lo"], case["n_hi"]), rng.choice(BATCH_DIMS)) for _ in range(case["problems"])]


def _ball_eps(n, d, s):
    """The distance whose d-ball holds `s` of n uniform points (boundary losses ignored)."""
    vol = math.pi ** (d / 2) / math.gamma(d / 2 + 1)
    return float((s / max(n - 1, 1) / vol) ** (1.0 / d))


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    state = {"case": case}
    if case["kind"] == "batch":
        sizes = _mix(case)
        rows = int(1.1 * (1.0 + case["s"]) * sum(n for n, _ in sizes))
        state["pairs"] = torch.full((rows, 2), -1, dtype=torch.int32, device="cuda")
        state["points"] = [_points("uniform", n, d, gen) for n, d in sizes]
        state["eps"] = [_ball_eps(n, d, case["s"]) for n, d in sizes]
    else:
        state["points"] = _points(case["dist"], case["n"], case["d"], gen)
        state["eps"] = _distance(state["points"], case["s"])
    if case["kind"] == "join":
        rows = int(1.3 * (1.0 + case["s"]) * case["n"])
        state["pairs"] = torch.full((rows, 2), -1, dtype=torch.int32, device="cuda")
        state["d2"] = torch.full((rows,), -1.0, dtype=torch.float64, device="cuda") if case["d2"] else None
    return state


def run(state):
    case, points, eps = state["case"], state["points"], state["eps"]
    kind, path = case["kind"], case["path"]
    if kind == "join":
        g = selfjoin_build_grid(points, eps)
        total, _, _ = selfjoin_count(g, path)
        written, cursor, _ = selfjoin_pairs(g, path, 0, state["pairs"], state["d2"])
        selfjoin_free_grid(g)
        out = {"total": total, "written": written, "cursor": cursor, "pairs": state["pairs"]}
        return dict(out, d2=state["d2"]) if case["d2"] else out
    if kind == "count":
        g = selfjoin_build_grid(points, eps, index_dims=case["index_dims"])
        total, per_point, _ = selfjoin_count(g, path, per_point=True)
        selfjoin_free_grid(g)
        return {"total": total, "per_point": per_point}
    if kind == "core":
        g = selfjoin_build_grid(points, eps, symmetric=1)
        flags, ncore = selfjoin_core_points(g, case["min_pts"], path)
        selfjoin_free_grid(g)
        return {"flags": flags, "ncore": ncore}
    if kind == "knn":
        g = selfjoin_build_grid(points, eps)
        nbr, d2, found = selfjoin_knn(g, case["k"], path)
        selfjoin_free_grid(g)
        return {"nbr": nbr, "d2": d2, "nfound": found}
    if kind == "noalloc":
        total, per_point = selfjoin_count_noalloc(points, eps, path, per_point=True)
        return {"total": total, "per_point": per_point}
    b = selfjoin_batch_build(points, eps)
    totals, _ = selfjoin_batch_count(b, path)
    offsets, _ = selfjoin_batch_pairs(b, path, state["pairs"])
    selfjoin_batch_free(b)
    return {"totals": torch.tensor(totals), "offsets": torch.tensor(offsets), "pairs": state["pairs"]}


def _work_one(n, d, s, pair_bytes, point_bytes, every=False):
    """Points read once, results written once; and of the arithmetic what no index can leave out: one distance
    (a subtraction and a multiply-add per dimension) for each unordered pair of the result, or for each of all
    unordered pairs where the mode asks for them (`every`)."""
    result = n * (1.0 + s)
    unordered = 0.5 * n * n if every else 0.5 * n * s
    return 8.0 * n * d + point_bytes * n + pair_bytes * result, 3.0 * d * unordered


def work(case):
    kind, s = case["kind"], case["s"]
    if kind == "batch":
        parts = [_work_one(n, d, s, 8, 0) for n, d in _mix(case)]
        return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}
    n, d = case["n"], case["d"]
    if kind == "join":
        b, f = _work_one(n, d, s, 16 if case["d2"] else 8, 0)
    elif kind == "core":
        b, f = _work_one(n, d, s, 0, 1)
    elif kind == "knn":
        b, f = _work_one(n, d, s, 0, 12 * case["k"] + 4)
    else:
        b, f = _work_one(n, d, s, 0, 4, every=case.get("index_dims") == -1)
    return {"bytes": b, "flops": f}


def exact(case, seed):
    """The squared distances of the neighbour lists in 64 bits. The other outputs are whole numbers, or distances
    in the order of the pair list, which is the library's own."""
    if case["kind"] != "knn":
        return None
    state = prepare(case, seed)
    points, eps, k = state["points"], state["eps"], case["k"]
    n, d = points.shape
    order = torch.argsort(points[:, 0])
    rows = points[order].contiguous()
    x = rows[:, 0].contiguous()
    out = torch.empty((n, k), dtype=torch.float64, device="cuda")
    step = 2048
    lows = torch.searchsorted(x, x[::step] - 1.001 * eps).tolist()
    lasts = torch.arange(step - 1, n + step - 1, step, device="cuda").clamp_(max=n - 1)
    highs = torch.searchsorted(x, x[lasts] + 1.001 * eps, right=True).tolist()
    for b, at in enumerate(range(0, n, step)):
        end, lo, hi = min(n, at + step), lows[b], highs[b]
        d2 = torch.zeros((end - at, hi - lo), dtype=torch.float64, device="cuda")
        for t in range(d):
            d2.add_((rows[at:end, t, None] - rows[None, lo:hi, t]).square_())
        own = torch.arange(end - at, device="cuda")
        d2[own, own + (at - lo)] = math.inf
        d2.masked_fill_(d2 > eps * eps, math.inf)
        kk = min(k, hi - lo)
        best = torch.topk(d2, kk, dim=1, largest=False, sorted=True).values
        out[at:end] = math.inf
        out[at:end, :kk] = best
    res = torch.empty_like(out)
    res[order] = out
    return {"nbr": None, "d2": res, "nfound": None}
