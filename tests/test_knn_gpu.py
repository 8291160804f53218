"""kNN selection around the sizes at which it changes its form (pairs of a
point: one wave's worth, the LDS form's limit) with equal distances and
duplicate points, against the oracle's lists."""
import numpy as np
import pytest

from tests.gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2209_11287_amd as p
    p.load()
    yield


@pytest.mark.parametrize("k", [1, 5, 64])
@pytest.mark.parametrize("ties", [True, False])
def test_group_sizes_around_the_limits(k, ties):
    import torch

    import oracle
    from paper_2209_11287_amd import SelfJoin
    rng = np.random.default_rng(k)
    # groups far apart, every pair of a group within eps: group size = pairs of each of its points
    X = []
    for c, m in enumerate([1, 2, 3, 4, 5, 63, 64, 65, 66, 128, 255, 256, 257, 258, 300]):
        off = rng.integers(0, 4, (m, 2)) / 64.0 if ties else rng.random((m, 2)) * 0.05
        X.append(off + [2.0 * c, 0.5 * c])
    X = np.concatenate(X)
    X = X[rng.permutation(len(X))]
    eps = 0.125
    want_nbr, want_d2, want_found = oracle.knn_within_eps(X, eps, k)
    log(f"[knn] groups k={k} ties={ties} n={len(X)}")
    sj = SelfJoin(torch.from_numpy(X).to("cuda:0"), eps)
    try:
        for budget in (0, 1000):
            nbr, d2, found = sj.knn(k, "fp64_mfma", pair_budget=budget)
            assert np.array_equal(found.cpu().numpy(), want_found)
            assert np.array_equal(nbr.cpu().numpy(), want_nbr)
            assert np.array_equal(d2.cpu().numpy(), want_d2)
    finally:
        sj.close()
