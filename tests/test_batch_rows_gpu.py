"""Rows, norms and offsets of a batched build at the edges of its blocks:
dimensions around the rows that one staged part holds, point counts around a
block of 256 rows and around a step of the offsets' scan, all in one batch.
Totals and pair sets against the oracle."""
import numpy as np
import pytest

from tests.gpu_util import log, pair_keys

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2209_11287_amd as p
    p.load()
    yield


@pytest.mark.parametrize("dims", [[1, 2, 3, 4], [5, 7, 8, 16, 17], [33, 63, 64, 65, 72], [128, 255, 256]])
def test_sizes(dims):
    import torch

    import oracle
    from paper_2209_11287_amd import (selfjoin_batch_build, selfjoin_batch_count, selfjoin_batch_free,
                                      selfjoin_batch_pairs)
    rng = np.random.default_rng(dims[0])
    X, eps = [], []
    for n in (1, 2, 63, 191, 192, 193, 255, 256, 257, 2047, 2048, 2049):
        for d in dims:
            if d > 64 and n > 257:
                continue
            X.append(rng.random((n, d)))
            eps.append(0.35 * np.sqrt(d / 6.0) * (1.0 if d > 2 else 0.05))
    want = [oracle.grid_pairs(x, e) for x, e in zip(X, eps)]
    rows = sum(w[0] for w in want)
    log(f"[batch rows] dims={dims} problems={len(X)} pairs={rows}")
    pairs = torch.empty((max(rows, 1), 2), dtype=torch.int32, device="cuda:0")
    b = selfjoin_batch_build([torch.from_numpy(x).to("cuda:0") for x in X], eps)
    try:
        totals, _ = selfjoin_batch_count(b, "fp64_mfma")
        offsets, _ = selfjoin_batch_pairs(b, "fp64_mfma", pairs)
        torch.cuda.synchronize()
    finally:
        selfjoin_batch_free(b)
    got = pairs.cpu().numpy()
    assert [int(t) for t in totals] == [w[0] for w in want]
    for k, w in enumerate(want):
        o = int(offsets[k])
        assert np.array_equal(pair_keys(got[o:o + w[0]]), pair_keys(w[2])), (k, X[k].shape)
