"""The allocation-free count at its limit: the largest sizes that it accepts run
within the static scratch (a buffer that did not fit would give a capacity
status in the middle of the call), with few and with many cells."""
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


def _accepts(x, eps):
    from paper_2209_11287_amd import SelfJoinError, selfjoin_count_noalloc
    from paper_2209_11287_amd._lib import SJ_ERR_CAPACITY
    try:
        return selfjoin_count_noalloc(x, eps, "fp64_mfma")[0]
    except SelfJoinError as e:
        assert e.status == SJ_ERR_CAPACITY and "scratch" in str(e)
        return None


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 8, 16, 17, 64, 65, 256])
def test_largest_accepted(d):
    import torch

    from paper_2209_11287_amd import SelfJoin
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(d)
    x = torch.rand((1_600_000 if d < 5 else 500_000, d), generator=gen, dtype=torch.float64, device="cuda:0")
    tiny = 1e-7  # as many cells as points
    lo, hi = 1, len(x)  # accepted; refused (before any device work)
    assert _accepts(x[:hi], tiny) is None
    while hi - lo > 1:
        mid = (lo + hi) // 2
        if _accepts(x[:mid], tiny) is None:
            hi = mid
        else:
            lo = mid
    log(f"[noalloc limit] d={d}: {lo} points")
    stated = {2: 1_290_000, 4: 647_000, 64: 151_000, 256: 47_400}  # the header's, rounded
    if d in stated:
        assert abs(lo - stated[d]) <= 0.01 * stated[d]
    for n in (lo, int(0.9 * lo), int(0.7 * lo)):
        for k in (0.02, 0.2):
            eps = float(k * n ** (-1.0 / d) * d ** 0.5) if d < 16 else k * 2.0
            sj = SelfJoin(x[:n], eps)
            want = sj.count("fp64_mfma")[0]
            sj.close()
            assert _accepts(x[:n], eps) == want
