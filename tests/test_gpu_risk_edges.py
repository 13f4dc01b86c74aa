"""Risk measures where the counted ranges end at the edges of the key space, against sorting the losses by their keys
(NaNs by sign: negative ones after every loss, positive ones before)."""
import numpy as np
import pytest

import oracle

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


# ---- ranks whose range is too large to copy out: rounds of bins over the whole grid
def _hard(n, kind):
    rng = np.random.default_rng(n + sum(map(ord, kind)))
    y = rng.lognormal(13, 2.2, size=n)
    seen = np.zeros(n, bool)
    seen[_sampled(n)] = True
    unseen = np.flatnonzero(~seen)
    if kind == "cluster":           # half of the losses close together, every one distinct
        at = rng.permutation(n)[: n // 2]
        y[at] = 1e7 * (1.0 + 1e-7 * rng.random(at.size))
    elif kind == "shared":          # the same, of three losses
        at = rng.permutation(n)[: n // 2]
        y[at] = np.nextafter(1e7, np.inf) * np.array([1.0, 1.0 + 2.0 ** -50, 1.0 + 2.0 ** -40])[np.arange(at.size) % 3]
    elif kind == "outlier":         # bins stretched by one loss over close ones
        y = 1e6 * (1.0 + 1e-4 * rng.random(n))
        y[n // 3] = 1e14
    elif kind == "unseen_top":      # far more keys below the smallest one sampled than are copied out
        y[unseen[: n // 2]] *= 1e6
    elif kind == "unseen_rest":     # the sample's own losses are the largest: the bins end before the ranks
        y[unseen] = 1.0 + rng.random(unseen.size)
        y[seen] = 1e9 + rng.random(int(seen.sum()))
    elif kind == "unseen_negative":  # zeros and negative losses that no sample shows
        y[unseen] = -1.0 - rng.random(unseen.size)
        y[unseen[: n // 4]] = 0.0
    elif kind == "around_zero":
        y = rng.normal(size=n)
    return y


def _check(y, rps, pml, tvar, what):
    order = np.sort(y + 0.0)[::-1]
    for rp, p, t in zip(rps, pml, tvar):
        k = oracle.rank(len(y), rp)
        assert p == order[k - 1], (what, rp, p, order[k - 1])
        # two orders of a k-term sum
        assert abs(t - order[:k].mean()) <= 2.0 * k * 2.0 ** -53 * np.abs(order[:k]).mean() + 1e-300, (what, rp)


HARD = ("cluster", "shared", "outlier", "unseen_top", "unseen_rest", "unseen_negative", "around_zero")


@pytest.mark.parametrize("kind", HARD)
@pytest.mark.parametrize("n", (16_385, 40_000, 700_001))
def test_ranges_too_large_to_copy(ara_lib, gpu_ctx, n, kind):
    import torch
    A = ara_lib
    print(f"risk large ranges n={n} {kind}", flush=True)
    y = _hard(n, kind)
    yt = torch.from_numpy(y).cuda()
    few = [1.0, 2.0, 3.0, 10.0, 100.0, float(n)]
    many = few + list(np.geomspace(1.1, n / 3.0, 14))          # two groups of ranks in one workspace
    for rps in (few, many):
        pml, tvar = A.ara_risk_measures(gpu_ctx, yt, rps)
        _check(y, rps, pml, tvar, (n, kind))
        if n <= A.ARA_NOALLOC_MAX_N:
            p2, t2 = A.ara_risk_measures_noalloc(gpu_ctx, yt, rps)
            assert p2.tobytes() == pml.tobytes() and t2.tobytes() == tvar.tobytes()


@pytest.mark.parametrize("n", (4_194_304, 4_194_305, 9_000_001))
def test_long_ylt(ara_lib, gpu_ctx, n):
    """Both samples, ranks of long return periods among the keys below the sampled ones."""
    import torch
    A = ara_lib
    print(f"risk long n={n}", flush=True)
    y = np.random.default_rng(n).lognormal(13, 2.2, size=n)
    rps = [2.0, 10.0, 250.0, 1000.0, 2000.0, 5000.0, float(n)]
    pml, tvar = A.ara_risk_measures(gpu_ctx, torch.from_numpy(y).cuda(), rps)
    _check(y, rps, pml, tvar, n)


def test_batch_with_large_ranges(ara_lib, gpu_ctx):
    """Some YLTs of a batch need further rounds, some do not; one set of launches and several."""
    import torch
    import synth
    from paper_1308_2066_amd import session
    A = ara_lib
    rng = np.random.default_rng(9)
    n, C = 40_000, 3_000
    ids, offs = synth.yet_poisson(rng, n, 3.0, C)
    an = session.open_analysis(gpu_ctx, ids, offs, C, [synth.elt_sparse(rng, 900, C, 10.0, 2.0)],
                               (1e3, 1e6, 1e4, 2e6))
    kinds = ("cluster", None, "unseen_top", "unseen_rest", None)
    lens = [n, n, n, 17_000, 9_000]
    ylts = [torch.empty(k, dtype=torch.float64, device="cuda") for k in lens]
    batch = A.ara_batch_create(gpu_ctx, [(an.yet, an.layer, 0, k, y) for k, y in zip(lens, ylts)])
    try:
        A.ara_batch_run(batch)
        host = []
        for y, kind, k in zip(ylts, kinds, lens):
            h = _hard(k, kind or "plain")
            y.copy_(torch.from_numpy(h))
            host.append(h)
        for rps in ([2.0, 10.0, 100.0], list(np.geomspace(1.0, 500.0, 33)), [2.0, 10.0, 100.0]):
            pml, tvar = A.ara_batch_risk(batch, rps)
            for j, h in enumerate(host):
                _check(h, rps, pml[j], tvar[j], (j, len(rps)))
    finally:
        A.ara_batch_release(batch)
        an.release()


def test_server_with_large_ranges(ara_lib, gpu_ctx):
    """Requests whose year losses are close together (one occurrence a year of an event of about 10^7), among others."""
    import torch
    from paper_1308_2066_amd import session
    A = ara_lib
    rng = np.random.default_rng(12)
    n, C = 60_000, 4_000
    ids = rng.integers(0, C, size=n).astype(np.int32)
    offs = np.arange(n + 1, dtype=np.int64)
    yet = A.ara_yet_create(gpu_ctx, session.to_device(ids), session.to_device(offs), C)
    close = 1e7 * (1.0 + 1e-9 * rng.random(C))
    close[: C // 4] = rng.lognormal(13, 2.2, size=C // 4)
    apart = rng.lognormal(13, 2.2, size=C)
    pool = [A.ara_elt_create(gpu_ctx, session.to_device(np.arange(C, dtype=np.int32)), session.to_device(v), C)
            for v in (close, apart)]
    rps = [2.0, 3.0, 10.0]
    srv = A.ara_server_create(gpu_ctx, yet, pool, rps, max_batch=4, memory_budget=1 << 28)
    try:
        inf = float("inf")
        asked = [([k % 2], (0.0, inf, 0.0, inf), 100 * k, n - 500 * k) for k in range(12)]
        tickets = [A.ara_server_submit(srv, *r) for r in asked]
        for (idx, _, t0, t1), t in zip(asked, tickets):
            pml, tvar = A.ara_server_wait(srv, t)[:2]
            _check((close, apart)[idx[0]][ids[t0:t1]], rps, pml, tvar, (idx, t0, t1))
    finally:
        A.ara_server_release(srv)
        for e in pool:
            A.ara_elt_release(e)
        A.ara_yet_release(yet)


def test_large_ranges_use_the_whole_grid(ara_lib, gpu_ctx):
    """Losses half of which are close take a few launches more than distinct ones (twice the time), not a walk by one
    workgroup (fifty times)."""
    import time
    import torch
    A = ara_lib
    n, took = 1_000_000, {}
    ws = torch.empty(A.ara_sort_workspace_size(n), dtype=torch.uint8, device="cuda")
    for kind in ("plain", "cluster"):
        y = torch.from_numpy(_hard(n, kind)).cuda()
        times = []
        for _ in range(15):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            A.ara_risk_measures(gpu_ctx, y, [10.0], ws)
            times.append(time.perf_counter() - t0)
        took[kind] = sorted(times)[7]
    assert took["cluster"] < 10.0 * took["plain"], took
