"""Hit-list count (d = 5 .. 64): pair lists in the order that the mask
expansion of the vector-ALU path gives (query order, then candidate order),
counts and distances, on every K-step count and its neighbours, ragged last
items, split walks, points whose bins are longer than a wave's and a block's
window, and a list that outgrows its first guess."""
import numpy as np
import pytest

from tests.gpu_util import gpu_join, log
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


def _eps(X, s):
    Y = X[:2000]
    d2 = ((X[:64, None, :] - Y[None]) ** 2).sum(2).ravel()
    return float(np.sqrt(np.partition(d2, int(64 + 64 * s * len(Y) / len(X)))[int(64 + 64 * s * len(Y) / len(X))]))


def _same(X, eps, path, capacity=None, **kw):
    import oracle
    log(f"[hits] path={path} n={X.shape[0]} d={X.shape[1]} eps={eps} capacity={capacity} {kw}")
    a = gpu_join(X, eps, path, want_d2=True, capacity=capacity, **kw)
    b = gpu_join(X, eps, "fp64_valu", want_d2=True, **kw)  # masks, exact chain
    total, pp, _, _ = oracle.grid_count(X, eps)
    assert a["total"] == b["total"] == total
    assert np.array_equal(a["per_point"], pp)
    assert np.array_equal(a["pairs"], b["pairs"])
    assert np.array_equal(a["d2"], b["d2"])
    return a


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("d", [5, 7, 8, 9, 12, 13, 16, 17, 20, 25, 31, 32, 36, 41, 47, 48, 53, 60, 63, 64])
def test_every_k_step_count(path, d):
    X = gen.gaussian_mixture(9007, d, clusters=6, seed=d)
    eps = _eps(X, 30)
    _same(X, eps, path)
    _same(X, eps, path, index_dims=1, short_circuit=-1)  # long lines, no box test


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("n", [2800, 2944, 2945, 2959, 2960, 2961, 3007, 3009])
def test_ragged_ends_and_smallest_work(path, n):
    # around whole blocks of 64 and tiles of 16 points; 2800 stays on the
    # per-wave tiles (less work than this count takes)
    X = gen.make("uniform", n, 6, seed=n)
    _same(X, 0.2, path, index_dims=-1)


@pytest.mark.parametrize("path", PATHS)
def test_chunks_and_skewed_points(path):
    X = gen.make("expo", 20011, 5, seed=3)
    _same(X, _eps(X, 40), path, capacity=50021)


@pytest.mark.parametrize("path", PATHS)
def test_long_bins_and_list_growth(path):
    # 1500 points at one place (more neighbours than a wave orders), a
    # spread set around them; then a set in which all 3000 points pair (the
    # list outgrows its first guess and the pairs call makes it again)
    rng = np.random.default_rng(2)
    X = np.concatenate([np.full((1500, 8), 0.25), rng.random((9000, 8))])[rng.permutation(10500)]
    _same(X, 0.3, path)
    _same(rng.random((3000, 6)) * 1e-3, 1.0, path)


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("scale", [2.0 ** -400, 1e100])
def test_units_far_from_one(path, scale):
    X = gen.gaussian_mixture(6001, 9, clusters=4, seed=4) * scale
    _same(X, _eps(X / scale, 25) * scale, path)


@pytest.mark.parametrize("symmetric", [0, 1])
@pytest.mark.parametrize("dims", [(8, 16, 5), (2, 8, 3, 16, 20)])
def test_batch_lists_equal_mask_expansion(symmetric, dims):
    """A batch with (and without) problems that stay on the per-wave tiles:
    pairs, offsets and totals of the hit-list count equal those that the
    vector-ALU path's masks give, in order; repeated counts; and a count on one
    path with the pairs asked for on the other."""
    import torch
    from paper_2209_11287_amd import (selfjoin_batch_build, selfjoin_batch_count, selfjoin_batch_free,
                                      selfjoin_batch_pairs)
    rng = np.random.default_rng(11)
    sizes = [0, 1, 65, 3000, 4511, 2500, 700]
    X = [rng.random((sizes[k % 7], dims[k % len(dims)])) for k in range(12)]
    X.append(rng.random((2500, dims[0])) * 1e-3)  # every pair within eps: the list outgrows its first guess
    eps = [0.1 * x.shape[1] ** 0.5 for x in X]
    pts = [torch.from_numpy(x).to("cuda:0") for x in X]

    def run(count_path, pairs_path, sym):
        b = selfjoin_batch_build(pts, eps, symmetric=sym)
        t0, _ = selfjoin_batch_count(b, count_path)
        t1, _ = selfjoin_batch_count(b, count_path)
        buf = torch.full((sum(t1) + 7, 2), -1, dtype=torch.int32, device="cuda:0")
        offs, _ = selfjoin_batch_pairs(b, pairs_path, buf)
        again = torch.full_like(buf, -1)
        selfjoin_batch_pairs(b, pairs_path, again)
        selfjoin_batch_free(b)
        assert t0 == t1 and torch.equal(buf, again)
        return t1, offs, buf.cpu().numpy()

    want = run("fp64_valu", "fp64_valu", 0)
    for cp, pp in (("fp64_mfma", "fp64_mfma"), ("fp64_mfma", "fp64_valu"), ("fp64_valu", "fp64_mfma")):
        log(f"[hits] batch dims={dims} symmetric={symmetric} count {cp} pairs {pp}")
        got = run(cp, pp, symmetric)
        assert got[0] == want[0] and got[1] == want[1]
        assert np.array_equal(got[2], want[2])


@pytest.mark.parametrize("n,d", [(140001, 5), (150016, 7)])
def test_long_walks_dealt_to_several_blocks(n, d):
    """Enough block items and rounds that the walks are split for evenness; per-point counts and the pair list
    against the vector-ALU path, which walks no hit list."""
    import torch

    rng = np.random.default_rng(n)
    X = rng.random((n, d))
    eps = 0.5 * (8.0 / n) ** (1.0 / d)
    log(f"[hits] long walks n={n} d={d} eps={eps}")
    got = gpu_join(X, eps, "fp64_mfma", index_dims=-1)
    want = gpu_join(X, eps, "fp64_valu", index_dims=-1)
    assert got["total"] == want["total"]
    assert np.array_equal(got["per_point"], want["per_point"])
    assert np.array_equal(got["pairs"], want["pairs"])
    torch.cuda.synchronize()
