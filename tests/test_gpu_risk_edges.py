"""Risk measures where the counted ranges end at the edges of the key space, against sorting the losses by their keys
(NaNs by sign: negative ones after every loss, positive ones before)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _sampled(n, stretches=1024):
    """Places the selection samples: one in each equal stretch of the YLT."""
    t = np.arange(stretches, dtype=np.uint64)
    a, e = t * np.uint64(n) // np.uint64(stretches), (t + np.uint64(1)) * np.uint64(n) // np.uint64(stretches)
    h = (t * np.uint64(2654435761)) & np.uint64(0xFFFFFFFF)
    return (a + ((h * (e - a)) >> np.uint64(32)))[e > a].astype(np.int64)


def _descending(y):
    u = (y + 0.0).view(np.uint64)
    asc = np.where(u >> np.uint64(63) != 0, ~u, u | np.uint64(1 << 63))
    return y[np.argsort(~asc, kind="stable")]


@pytest.mark.parametrize("n", (5_000, 16_384, 16_385, 40_000))
def test_rank_among_negative_nans(ara_lib, gpu_ctx, n):
    """The first negative NaN is a rank, its bin ends with the key space, and positive NaNs that no sample shows are
    the smallest keys: they are not in that bin."""
    import torch
    A = ara_lib
    print(f"risk negative NaNs n={n}", flush=True)
    neg = np.array([0xFFFFFFFFFFFFFFFF], np.uint64).view(np.float64)[0]
    y = np.full(n, 2.0 ** 20)
    y[::3] = neg
    y[1::10] = 3.0
    unseen = np.setdiff1d(np.arange(n), _sampled(n))[:: max(1, n // 40)]
    y[unseen] = np.nan
    order = _descending(y)
    count = int(np.sum(np.isnan(y) & np.signbit(y)))
    ks = [n - count + 1, n, n // 2]
    rps = [n / k for k in ks]
    pml, tvar = A.ara_risk_measures(gpu_ctx, torch.from_numpy(y).cuda(), rps)
    want = np.array([order[k - 1] for k in ks])
    assert np.array_equal(np.isnan(pml), np.isnan(want)) and np.array_equal(np.signbit(pml), np.signbit(want))
    assert pml[2] == want[2] and np.isnan(tvar).all()
