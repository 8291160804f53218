"""The rule that gives a count its list of pairs or the in-masks of all
candidates, the first layout of the list, and the list count where the rule
would not take it (many pairs a point): counts, pairs in order and distances."""
import ctypes

import numpy as np
import pytest

from tests.gpu_util import gpu_join, log, pair_keys
from workloads import generators as gen

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


class _hits:
    """List count always (where grid, path and work allow it), with `first`
    entries per region of the list's first layout (0: the library's)."""

    def __init__(self, first=0):
        from paper_2209_11287_amd import _lib
        self.f = _lib.load().sj_test_hits
        self.f.restype = None
        self.f.argtypes = [ctypes.c_int32, ctypes.c_ulonglong]
        self.first = first

    def __enter__(self):
        self.f(1, self.first)

    def __exit__(self, *exc):
        self.f(0, 0)


def _same(X, eps, path, first=0, **kw):
    import oracle
    log(f"[hits rule] path={path} n={X.shape[0]} d={X.shape[1]} eps={eps} first={first} {kw}")
    with _hits(first):
        a = gpu_join(X, eps, path, want_d2=True, **kw)
    kw.pop("capacity", None)
    b = gpu_join(X, eps, "fp64_valu", want_d2=True, **kw)  # in-masks, exact chain
    total, pp, _, _ = oracle.grid_count(X, eps)
    assert a["total"] == b["total"] == total
    assert np.array_equal(a["per_point"], pp)
    assert np.array_equal(a["pairs"], b["pairs"])
    assert np.array_equal(a["d2"], b["d2"])


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("symmetric", [0, 1])
def test_list_that_outgrows_its_first_layout(path, symmetric):
    X = gen.make("uniform", 9007, 8, seed=8)
    _same(X, 0.4, path, first=256, symmetric=symmetric)
    _same(X, 0.4, path, first=256, symmetric=symmetric, capacity=40009)


@pytest.mark.parametrize("path", PATHS)
def test_dense_sets_in_a_list(path):
    rng = np.random.default_rng(5)
    _same(rng.random((3000, 6)) * 1e-3, 1.0, path)  # every pair
    X = np.concatenate([np.full((1500, 8), 0.25), rng.random((9000, 8))])[rng.permutation(10500)]
    _same(X, 0.6, path)


@pytest.mark.parametrize("first", [0, 256])
def test_dense_batch_in_a_list(first):
    import torch

    import oracle
    from paper_2209_11287_amd import (selfjoin_batch_build, selfjoin_batch_count, selfjoin_batch_free,
                                      selfjoin_batch_pairs)
    rng = np.random.default_rng(6)
    X = [rng.random((n, d)) for n, d in ((3001, 5), (2500, 16), (1200, 3), (3000, 8))]
    X[0] *= 1e-3
    eps = [1.0, 1.5, 0.1, 0.5]
    log(f"[hits rule] dense batch first={first}")
    with _hits(first):
        b = selfjoin_batch_build([torch.from_numpy(x).to("cuda:0") for x in X], eps)
        totals, _ = selfjoin_batch_count(b, "fp64_mfma")
        buf = torch.full((sum(totals), 2), -1, dtype=torch.int32, device="cuda:0")
        offsets, _ = selfjoin_batch_pairs(b, "fp64_mfma", buf)
        selfjoin_batch_free(b)
    got = buf.cpu().numpy()
    for k, x in enumerate(X):
        want = oracle.grid_pairs(x, eps[k])[2]
        assert int(totals[k]) == len(want)
        o = int(offsets[k])
        assert np.array_equal(pair_keys(got[o:o + len(want)]), pair_keys(want)), k


def test_dense_set_keeps_in_masks():
    """Every pair within eps (20,000 neighbours a point): the count keeps the
    bit per candidate (about 50 MB) and no list (1.6 GB of pairs)."""
    import torch

    from paper_2209_11287_amd import SelfJoin
    n = 20000
    xt = torch.rand((n, 6), dtype=torch.float64, device="cuda:0") * 1e-3
    log("[hits rule] in-masks")
    sj = SelfJoin(xt, 1.0, torch_alloc=True)
    before = torch.cuda.memory_allocated()
    total, _, _ = sj.count("fp64_mfma")
    held = torch.cuda.memory_allocated() - before
    assert total == n * n
    assert n * n // 8 <= held <= n * n // 4
    buf = torch.empty((total, 2), dtype=torch.int32, device="cuda:0")
    assert torch.equal(sj.all_pairs("fp64_mfma")[:, 1].to(torch.int64).sum(), torch.tensor(n * n * (n - 1) // 2, device="cuda:0"))
    del buf
    sj.close()


@pytest.mark.parametrize("eps", [0.08, 0.09, 0.1])
@pytest.mark.parametrize("path", ["fp64_mfma", "fp32_mfma"])
def test_distances_asked_for_at_once(path, eps):
    """A pairs call with distances (56, 148 and 303 pairs a point) and without a
    count before it takes the list further than a count does."""
    import torch

    from paper_2209_11287_amd import SelfJoin, selfjoin_pairs
    X = torch.from_numpy(gen.gaussian_mixture(100000, 16, seed=3)).to("cuda:0")
    log(f"[hits rule] distances at once path={path} eps={eps}")
    out = []
    for counted in (True, False):
        sj = SelfJoin(X, eps)
        if counted:
            total = sj.count(path)[0]
        pairs = torch.empty((total, 2), dtype=torch.int32, device="cuda:0")
        d2 = torch.empty(total, dtype=torch.float64, device="cuda:0")
        assert selfjoin_pairs(sj.grid, path, 0, pairs, d2)[0] == total
        sj.close()
        out.append((pairs, d2))
    (a, ad), (b, bd) = out
    assert torch.equal(a, b) and torch.equal(ad, bd)


def test_large_set_keeps_its_list():
    """33.6M points one unit apart on a line, 3 pairs a point: a first layout of
    256 pairs a point would pass the list's budget, the list itself does not. At
    this size the pairs are placed one by one (buckets hold fewer points) and the
    tables' tile sums are scanned by a launch of their own."""
    import torch

    from paper_2209_11287_amd import SelfJoin, selfjoin_pairs
    n = 33_600_000
    dev = "cuda:0"
    at = torch.randperm(n, device=dev)  # place of each input row
    x = torch.zeros((n, 5), dtype=torch.float64, device=dev)
    x[:, 3] = at
    log(f"[hits rule] line of {n} points")
    with _hits():
        sj = SelfJoin(x, 1.5, torch_alloc=True)
        before = torch.cuda.memory_allocated()
        total, pp, _ = sj.count("fp64_mfma", per_point=True)
        assert torch.cuda.memory_allocated() - before > 1 << 30  # (without a list 0.6 GiB)
        assert total == 3 * n - 2
        assert int((pp == 3).sum()) == n - 2 and int((pp == 2).sum()) == 2
        buf = torch.empty((total, 2), dtype=torch.int32, device=dev)
        written = selfjoin_pairs(sj.grid, "fp64_mfma", 0, buf)[0]
        sj.close()
    assert written == total
    q, c = at[buf[:, 0].long()], at[buf[:, 1].long()]
    del buf, x, sj
    # queries by place, each with the place before, its own and the one after
    k = torch.arange(1, total + 1, device=dev)
    assert torch.equal(q, k // 3)
    assert torch.equal(c - q, k % 3 - 1)
    del q, c, k, at, pp
    torch.cuda.empty_cache()


# The list count's own tests with the rule set aside (in-masks would be taken for
# some of their sets).

@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("d", [5, 7, 8, 9, 12, 13, 16, 17, 20, 25, 31, 32, 36, 41, 47, 48, 53, 60, 63, 64])
def test_every_k_step_count_in_a_list(path, d):
    from tests import test_hits_gpu as t
    with _hits():
        t.test_every_k_step_count(path, d)


@pytest.mark.parametrize("path", PATHS)
def test_skewed_and_far_units_in_a_list(path):
    from tests import test_hits_gpu as t
    with _hits():
        t.test_chunks_and_skewed_points(path)
        for scale in (2.0 ** -400, 1e100):
            t.test_units_far_from_one(path, scale)


@pytest.mark.parametrize("symmetric", [0, 1])
@pytest.mark.parametrize("dims", [(8, 16, 5), (2, 8, 3, 16, 20)])
def test_batch_in_a_list(symmetric, dims):
    from tests import test_hits_gpu as t
    with _hits():
        t.test_batch_lists_equal_mask_expansion(symmetric, dims)
