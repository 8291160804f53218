"""Hit-list count on lattices, where many pairs lie at eps itself and every
path has to decide them with the exact chain: counts, pairs and distances
against the oracle, and that FP64 tiles did recheck pairs. Also walks that are
dealt to several blocks, against the oracle."""
import functools

import numpy as np
import pytest

from tests.gpu_util import gpu_join, log, pair_keys
from tests.test_hits_rule_gpu import _hits

pytestmark = pytest.mark.gpu

PATHS = ["fp64_mfma", "fp32_mfma", "bf16x3_mfma"]


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2209_11287_amd as p
    p.load()
    yield


def _lattice(kind):
    rng = np.random.default_rng(7)
    if kind == "cube5":    # 6^5 points, pairs two steps apart on one axis or one step on four
        g = np.arange(6.0)
        X = np.stack(np.meshgrid(g, g, g, g, g, indexing="ij"), -1).reshape(-1, 5)
        return X[rng.permutation(len(X))], 2.0
    if kind == "cube6":    # the same in steps of a tenth, which no binary fraction is
        g = 0.1 * np.arange(5)
        X = np.stack(np.meshgrid(*[g] * 6, indexing="ij"), -1).reshape(-1, 6)
        X = X[rng.permutation(len(X))[:9001]]
        return X, 0.2
    # random points of {0, 1, 2}^d in tenths
    d = int(kind[1:])
    return 0.1 * rng.integers(0, 3, (6001, d)), 0.1 * {8: 2.0, 16: 3.0, 33: 5.0, 64: 8.0}[d]


@functools.lru_cache(maxsize=None)
def _solved(kind):
    import oracle
    X, eps = _lattice(kind)
    return X, eps, oracle.grid_pairs(X, eps)[:3]


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("symmetric", [0, 1])
@pytest.mark.parametrize("kind", ["cube5", "cube6", "r8", "r16", "r33", "r64"])
def test_pairs_at_eps(kind, path, symmetric):
    X, eps, (total, pp, want) = _solved(kind)
    log(f"[hits ties] {kind} path={path} symmetric={symmetric} total={total}")
    with _hits():
        g = gpu_join(X, eps, path, want_d2=True, symmetric=symmetric)
    assert g["total"] == total and np.array_equal(g["per_point"], pp)
    assert np.array_equal(pair_keys(g["pairs"]), pair_keys(want))
    assert g["stats"]["rechecked"] > 0 and g["stats"]["rechecked_in"] > 0
    a, b = X[g["pairs"][:, 0]], X[g["pairs"][:, 1]]
    assert np.all(np.abs(((a - b) ** 2).sum(1) - g["d2"]) <= 1e-12 * eps * eps)
    assert np.all(g["d2"] <= eps * eps)


def test_batch_pairs_at_eps():
    import torch

    from paper_2209_11287_amd import (selfjoin_batch_build, selfjoin_batch_count, selfjoin_batch_free,
                                      selfjoin_batch_pairs)
    solved = [_solved(k) for k in ("cube5", "r16", "cube6", "r64")]
    sets = [(X, e) for X, e, _ in solved]
    want = [r[2] for _, _, r in solved]
    log(f"[hits ties] batch pairs={[len(w) for w in want]}")
    with _hits():
        b = selfjoin_batch_build([torch.from_numpy(X).to("cuda:0") for X, _ in sets], [e for _, e in sets])
        totals, st = selfjoin_batch_count(b, "fp64_mfma")
        buf = torch.full((sum(totals), 2), -1, dtype=torch.int32, device="cuda:0")
        offsets, _ = selfjoin_batch_pairs(b, "fp64_mfma", buf)
        selfjoin_batch_free(b)
    assert st["rechecked_in"] > 0
    got = buf.cpu().numpy()
    for k, w in enumerate(want):
        o = int(offsets[k])
        assert int(offsets[k + 1]) - o == len(w)
        assert np.array_equal(pair_keys(got[o:o + len(w)]), pair_keys(w)), k


@pytest.mark.parametrize("path", PATHS)
def test_long_walks_against_the_oracle(path):
    import oracle
    n, d = 140001, 5
    X = np.random.default_rng(n).random((n, d))
    eps = 0.5 * (8.0 / n) ** (1.0 / d)
    total, pp, want = oracle.grid_pairs(X, eps)[:3]
    log(f"[hits ties] long walks path={path} n={n} total={total}")
    with _hits():
        g = gpu_join(X, eps, path, index_dims=-1)
    assert g["total"] == total and np.array_equal(g["per_point"], pp)
    assert np.array_equal(pair_keys(g["pairs"]), pair_keys(want))
