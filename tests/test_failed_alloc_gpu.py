"""Calls after a failed device allocation (each failed once, on purpose, on the
host): the same handle goes on giving the oracle's results, and what the failed
call had allocated is given back."""
import ctypes

import numpy as np
import pytest

from tests.gpu_util import log, pair_keys
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


def _fail(nbytes, skip=0):
    from paper_2209_11287_amd import _lib
    f = _lib.load().sj_test_fail_alloc
    f.restype = None
    f.argtypes = [ctypes.c_size_t, ctypes.c_int32]
    f(int(nbytes), int(skip))


def _attempt(call):
    """The call's result, or None after an out-of-memory status."""
    from paper_2209_11287_amd import SelfJoinError
    from paper_2209_11287_amd._lib import SJ_ERR_OOM
    try:
        return call()
    except SelfJoinError as e:
        assert e.status == SJ_ERR_OOM
        return None
    finally:
        _fail(0)


def _points(n=9007, d=8, s=30):
    """Points with about s neighbours among many candidates: the calls that
    count into a list of pairs."""
    X = gen.make("uniform", n, d, seed=d)
    d2 = np.sort(((X[:64, None, :] - X[None]) ** 2).sum(2).ravel())
    return X, float(np.sqrt(d2[64 + 64 * s]))


@pytest.mark.parametrize("what", ["bins", "parts"])
def test_pairs_after_failed_bins(what):
    """The list by point (bins, 4 bytes a pair) or its first stage (parts, 8
    bytes a listed pair end) cannot be allocated."""
    import torch

    import oracle
    from paper_2209_11287_amd import SelfJoin, selfjoin_pairs
    X, eps = _points()
    total, _, want = oracle.grid_pairs(X, eps)[:3]
    xt = torch.from_numpy(X).to("cuda:0")
    held = torch.cuda.memory_allocated()
    sj = SelfJoin(xt, eps, torch_alloc=True)
    assert sj.count("fp64_mfma")[0] == total
    with_counts = torch.cuda.memory_allocated()
    log(f"[failed alloc] single {what} total={total}")
    for k in range(2):
        buf = torch.full((total, 2), -1, dtype=torch.int32, device="cuda:0")
        before = torch.cuda.memory_allocated()
        if k == 0:
            _fail(4 * total if what == "bins" else 8 * (total - len(X)))
        r = _attempt(lambda: selfjoin_pairs(sj.grid, "fp64_mfma", 0, buf))
        if k == 0 and r is None:
            assert torch.cuda.memory_allocated() == before
            assert before >= with_counts
            continue
        assert r[0] == total
        assert np.array_equal(pair_keys(buf.cpu().numpy()), pair_keys(want))
    del buf
    sj.close()
    torch.cuda.synchronize()
    assert torch.cuda.memory_allocated() == held


def _batch():
    import oracle
    sets = [_points(n, d) for n, d in ((4007, 8), (3001, 16), (2500, 3), (3500, 5))]
    want = [oracle.grid_pairs(X, e)[2] for X, e in sets]
    return sets, want


def _check_batch(offsets, buf, want):
    got = buf.cpu().numpy()
    for k, w in enumerate(want):
        o = int(offsets[k])
        assert int(offsets[k + 1]) - o == len(w)
        assert np.array_equal(pair_keys(got[o:o + len(w)]), pair_keys(w)), k


@pytest.mark.parametrize("what", ["bins", "parts"])
def test_batch_pairs_after_failed_bins(what):
    import torch

    from paper_2209_11287_amd import (selfjoin_batch_build, selfjoin_batch_count, selfjoin_batch_free,
                                      selfjoin_batch_pairs)
    sets, want = _batch()
    b = selfjoin_batch_build([torch.from_numpy(X).to("cuda:0") for X, _ in sets], [e for _, e in sets])
    totals, _ = selfjoin_batch_count(b, "fp64_mfma")
    assert [int(t) for t in totals] == [len(w) for w in want]
    listed = [(len(w), len(X)) for (X, _), w in zip(sets, want) if X.shape[1] > 4]
    pairs, rows = sum(p for p, _ in listed), sum(r for _, r in listed)
    log(f"[failed alloc] batch {what} listed pairs={pairs}")
    for k in range(2):
        buf = torch.full((sum(totals), 2), -1, dtype=torch.int32, device="cuda:0")
        if k == 0:
            _fail(4 * pairs if what == "bins" else 8 * (pairs - rows))
        r = _attempt(lambda: selfjoin_batch_pairs(b, "fp64_mfma", buf))
        if r is not None:
            _check_batch(r[0], buf, want)
        else:
            assert k == 0
    selfjoin_batch_free(b)


@pytest.mark.parametrize("path", ["fp64_mfma", "fp32_mfma", "bf16x3_mfma"])
def test_single_goes_on_without_the_list(path):
    """No memory for the list at the count, nor at the pairs call that would
    make it; then for the bins of a list that the pairs call has made: the tiles
    run again, and the statistics are theirs alone."""
    import torch

    import oracle
    from paper_2209_11287_amd import SelfJoin, selfjoin_pairs
    X, eps = _points()
    total, pp, want = oracle.grid_pairs(X, eps)[:3]
    xt = torch.from_numpy(X).to("cuda:0")
    log(f"[failed alloc] no list path={path} total={total}")

    def pairs(sj, **fail):
        buf = torch.full((total, 2), -1, dtype=torch.int32, device="cuda:0")
        if fail:
            _fail(**fail)
        r = selfjoin_pairs(sj.grid, path, 0, buf)
        _fail(0)
        assert r[0] == total and np.array_equal(pair_keys(buf.cpu().numpy()), pair_keys(want))
        return r[2]

    big = 1 << 22  # only the list is larger
    sj = SelfJoin(xt, eps)
    _fail(big)
    t, per_point, _ = sj.count(path, per_point=True)
    _fail(0)
    assert t == total and np.array_equal(per_point.cpu().numpy(), pp)
    tiles = pairs(sj, nbytes=big)  # no list again
    after_list = pairs(sj, nbytes=8 * (total - len(X)), skip=1)  # the list, then no parts
    assert (after_list["rechecked"], after_list["rechecked_in"]) == (tiles["rechecked"], tiles["rechecked_in"])
    pairs(sj)
    pairs(sj)
    sj.close()


def test_single_goes_on_without_the_index():
    import torch

    import oracle
    from paper_2209_11287_amd import SelfJoin
    X, eps = _points(9007, 48)
    total, pp, want = oracle.grid_pairs(X, eps)[:3]
    log(f"[failed alloc] no index total={total}")
    sj = SelfJoin(torch.from_numpy(X).to("cuda:0"), eps)
    _fail(2 * 48 * 4 * (len(X) // 16))  # the boxes
    t, per_point, _ = sj.count("fp64_mfma", per_point=True)
    _fail(0)
    assert t == total and np.array_equal(per_point.cpu().numpy(), pp)
    assert np.array_equal(pair_keys(sj.all_pairs("fp64_mfma").cpu().numpy()), pair_keys(want))
    sj.close()


@pytest.mark.parametrize("symmetric", [0, 1])
@pytest.mark.parametrize("pairs_path", ["fp64_mfma", "fp64_valu"])
def test_batch_goes_on_without_the_list(symmetric, pairs_path):
    """No memory for the batch's list at the count and at the pairs call: the
    tiles of its problems run again; with memory the list is made."""
    import torch

    from paper_2209_11287_amd import (selfjoin_batch_build, selfjoin_batch_count, selfjoin_batch_free,
                                      selfjoin_batch_pairs)
    sets, want = _batch()
    b = selfjoin_batch_build([torch.from_numpy(X).to("cuda:0") for X, _ in sets], [e for _, e in sets],
                             symmetric=symmetric)
    big = 1 << 22
    log(f"[failed alloc] batch without list symmetric={symmetric} pairs {pairs_path}")
    if not symmetric:
        _fail(big)
    totals, _ = selfjoin_batch_count(b, "fp64_mfma")
    _fail(0)
    assert [int(t) for t in totals] == [len(w) for w in want]
    for fail in (True, False):
        buf = torch.full((sum(totals), 2), -1, dtype=torch.int32, device="cuda:0")
        if fail:
            _fail(big)
        offsets, _ = selfjoin_batch_pairs(b, pairs_path, buf)
        _fail(0)
        _check_batch(offsets, buf, want)
    selfjoin_batch_free(b)


def test_count_after_a_failed_count():
    """The offsets could not be allocated: the next count makes them."""
    import torch

    import oracle
    from paper_2209_11287_amd import SelfJoin, SelfJoinError
    X, eps = _points(5000, 4)
    total, pp, want = oracle.grid_pairs(X, eps)[:3]
    log(f"[failed alloc] offsets total={total}")
    sj = SelfJoin(torch.from_numpy(X).to("cuda:0"), eps)
    _fail(8 * len(X))
    with pytest.raises(SelfJoinError):
        sj.count("fp64_valu")
    _fail(0)
    t, per_point, _ = sj.count("fp64_valu", per_point=True)
    assert t == total and np.array_equal(per_point.cpu().numpy(), pp)
    assert np.array_equal(pair_keys(sj.all_pairs("fp64_valu").cpu().numpy()), pair_keys(want))
    sj.close()
