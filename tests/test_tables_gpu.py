"""Grid tables and candidate ranges at the sizes where their kernels change:
around 64-point steps, tiles of several steps, lines of one point, lines that
cross steps and tiles, one long line, item counts around the groups of the
range search, with and without the dense line table."""
import numpy as np
import pytest

from tests.gpu_util import gpu_join, log, pair_keys
from workloads import generators as gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2209_11287_amd as p
    p.load()
    yield


def _check(X, eps, tag, pairs=True, **kw):
    import oracle
    total, pp, cref, _ = oracle.grid_count(X, eps)
    log(f"[tables] {tag} n={X.shape[0]} d={X.shape[1]} eps={eps} {kw}")
    g = gpu_join(X, eps, "fp64_mfma", want_pairs=pairs, **kw)
    assert g["total"] == total and np.array_equal(g["per_point"], pp)
    if not kw:
        assert g["info"]["cand_ref"] == cref
    if pairs:
        _, _, op = oracle.grid_pairs(X, eps)
        assert np.array_equal(pair_keys(g["pairs"]), pair_keys(op))
    # items: 16 points of one line, lines filled in order
    info = g["info"]
    assert info["items"] >= (info["n"] + 15) // 16 and info["cells"] <= info["n"]


@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 128, 255, 256, 257, 1023, 1025, 4096, 4097])
@pytest.mark.parametrize("d,k", [(1, 0), (2, 0), (3, 0), (4, 0), (3, 1)])
def test_ends_of_steps_and_lines(n, d, k):
    # wide cells: few long lines; narrow cells: about a line a point
    X = gen.make("uniform", n, d, seed=10 * n + d)
    for eps in (0.3, 0.5 / max(2, n) ** (1.0 / d)):
        _check(X, eps, "uniform", index_dims=k) if k else _check(X, eps, "uniform")


def test_no_line_table():
    # leading dimensions of 2^30 lines: the searches run over all rows
    rng = np.random.default_rng(1)
    X = np.concatenate([rng.random((3000, 3)), rng.random((50, 3)) * 2.0 ** 16])
    _check(X, 0.05, "wide")


@pytest.mark.parametrize("n,d", [(530001, 2), (700003, 4), (2200001, 3)])
def test_several_steps_per_wave(n, d):
    # more than one step of 64 a wave, and items beyond the range search's split
    X = gen.make("expo", n, d, seed=7)
    eps = 0.2 / 40 * (1.0 / n) ** (1.0 / d) * 8
    _check(X, eps, "expo", pairs=False)


@pytest.mark.parametrize("d", [2, 6])  # keys packed with their index; wide keys
@pytest.mark.parametrize("n", [63, 64, 65, 255, 257, 1023, 1024, 1025, 4095, 4096, 4097, 8193, (1 << 18) - 1,
                               1 << 18, (1 << 18) + 1])
def test_sort_tile_edges(n, d):
    """Whole and ragged tiles of both sizes, one digit holding most keys."""
    import oracle
    rng = np.random.default_rng(n + d)
    X = rng.random((n, d))
    X[: n // 2, 1:] *= 1e-3
    eps = 0.25 * n ** -0.5
    log(f"[sort] n={n} d={d}")
    total, pp, _, _ = oracle.grid_count(X, eps)
    g = gpu_join(X, eps, "fp64_mfma", want_pairs=False)
    assert g["total"] == total and np.array_equal(g["per_point"], pp)
