"""kNN selection of few neighbours among many pairs: around the sizes from
which it goes by rounds, with equal distances and without, against the oracle's
lists."""
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


@pytest.mark.parametrize("k", [1, 2, 3])
@pytest.mark.parametrize("ties", [True, False])
def test_few_neighbours_of_many(k, ties):
    """Around the group sizes from which few neighbours are taken in rounds
    (24 pairs for k = 1, 48 for k = 2, 60 for k = 3 at one part of 64)."""
    import torch

    import oracle
    from paper_2209_11287_amd import SelfJoin
    rng = np.random.default_rng(10 + k)
    X = []
    for c, m in enumerate([k, k + 1, 23, 24, 25, 47, 48, 49, 52, 53, 60, 61, 64, 65, 72, 73, 96, 97]):
        off = rng.integers(0, 4, (m, 2)) / 64.0 if ties else rng.random((m, 2)) * 0.05
        X.append(off + [2.0 * c, 0.5 * c])
    X = np.concatenate(X)
    X = X[rng.permutation(len(X))]
    want_nbr, want_d2, want_found = oracle.knn_within_eps(X, 0.125, k)
    log(f"[knn] few of many k={k} ties={ties} n={len(X)}")
    sj = SelfJoin(torch.from_numpy(X).to("cuda:0"), 0.125)
    try:
        nbr, d2, found = sj.knn(k, "fp64_mfma")
        assert np.array_equal(found.cpu().numpy(), want_found)
        assert np.array_equal(nbr.cpu().numpy(), want_nbr)
        assert np.array_equal(d2.cpu().numpy(), want_d2)
    finally:
        sj.close()
