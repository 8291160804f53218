"""The candidate pairs a hit-list count reports are those it met: of an
index-free set every unordered pair of blocks of 64 points once, and each
block with itself."""
import numpy as np
import pytest

from tests.gpu_util import gpu_join, log
from tests.test_hits_rule_gpu import _hits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2209_11287_amd as p
    p.load()
    yield


def _met(n):
    rows = [64] * (n // 64) + ([n % 64] if n % 64 else [])
    return (n * n + sum(r * r for r in rows)) // 2


@pytest.mark.parametrize("path", ["fp64_mfma", "fp32_mfma", "bf16x3_mfma"])
@pytest.mark.parametrize("n,sc,symmetric", [(6400, -1, 0), (6401, 0, 0), (9007, 0, 1), (70001, 0, 0)])
def test_pairs_met(path, n, sc, symmetric):
    rng = np.random.default_rng(n)
    X = rng.random((n, 8))
    log(f"[hits stats] path={path} n={n} sc={sc} symmetric={symmetric}")
    with _hits():
        st = gpu_join(X, 0.2, path, want_pairs=False, index_dims=-1, short_circuit=sc, symmetric=symmetric)["stats"]
    assert st["cand_eval"] == _met(n)
    if sc == -1 or path != "fp64_mfma":
        assert st["tiles_pruned"] == 0


@pytest.mark.parametrize("symmetric", [0, 1])
def test_batch_counts_each_form(symmetric):
    """Problems with a hit list and without one, together: what each problem
    alone reports."""
    import torch

    from paper_2209_11287_amd import SelfJoin, selfjoin_batch_build, selfjoin_batch_count, selfjoin_batch_free
    rng = np.random.default_rng(4)
    sets = [(rng.random((9001, 8)), 0.3), (rng.random((4000, 3)), 0.1), (rng.random((7000, 6)), 0.25)]
    pts = [torch.from_numpy(x).to("cuda:0") for x, _ in sets]
    with _hits():  # (a batch may choose otherwise than each problem alone)
        alone = {"fp64_mfma": 0, "fp64_valu": 0}
        for (x, e), p in zip(sets, pts):
            sj = SelfJoin(p, e, symmetric=symmetric)
            for path in alone:
                alone[path] += sj.count(path)[2]["cand_eval"]
            sj.close()
        assert alone["fp64_mfma"] != alone["fp64_valu"]  # a hit list was kept
        b = selfjoin_batch_build(pts, [e for _, e in sets], symmetric=symmetric)
        log(f"[hits stats] batch symmetric={symmetric}")
        for path in ("fp64_mfma", "fp64_valu", "fp64_mfma"):
            assert selfjoin_batch_count(b, path)[1]["cand_eval"] == alone[path]
        selfjoin_batch_free(b)
