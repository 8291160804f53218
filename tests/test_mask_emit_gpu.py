"""Pairs from the in-masks at full and ragged groups: every candidate of a
16-tile group a pair (256 places per query), the sizes around a group's end,
and sparse rows, with and without distances, on the d <= 4 form and the
general one; chunks that cut an item. Pair sets and distances against the
oracle; a distance is the dim-ascending FMA chain, so it is compared exactly."""
import numpy as np
import pytest

from tests.gpu_util import gpu_join, log, pair_keys

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2209_11287_amd as p
    p.load()
    yield


@pytest.mark.parametrize("d", [1, 3, 4, 6])
@pytest.mark.parametrize("n", [15, 16, 17, 255, 256, 257, 513, 1025])
@pytest.mark.parametrize("dense", [True, False])
def test_groups(n, d, dense):
    import oracle
    rng = np.random.default_rng(1000 * d + n)
    # lattice coordinates: squared distances are exact, so the chain's order cannot matter
    X = rng.integers(0, 8 if dense else 64, (n, d)) / 64.0
    eps = 0.125 * np.sqrt(d) if dense else 0.125
    total, pp, op = oracle.grid_pairs(X, eps)
    for capacity in (None, max(1, total // 3)):
        for d2 in (True, False):
            log(f"[mask emit] n={n} d={d} dense={dense} d2={d2} capacity={capacity} total={total}")
            g = gpu_join(X, eps, "fp64_mfma", want_d2=d2, capacity=capacity)
            assert g["total"] == total and np.array_equal(g["per_point"], pp)
            assert np.array_equal(pair_keys(g["pairs"]), pair_keys(op))
            if d2:
                i, j = g["pairs"][:, 0], g["pairs"][:, 1]
                assert np.array_equal(g["d2"], ((X[i] - X[j]) ** 2).sum(1))
