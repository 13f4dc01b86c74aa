"""ara_sort_desc at the sizes where its path changes (one workgroup, sampled buckets, radix passes), on distinct,
repeated, signed and special values, in place, and on a sample that misses almost every loss (a bucket past LDS).
The order is exact: the sorted values are the inputs' bits, -0.0 as +0.0."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _sorted(x):
    u = (x + 0.0).view(np.uint64)
    key = np.where(u >> np.uint64(63) != 0, ~u, u | np.uint64(1 << 63))
    return (x + 0.0)[np.argsort(~key, kind="stable")]


def _values(kind, n, rng):
    if kind == "distinct":
        return rng.lognormal(10, 2, n)
    if kind == "few":
        return rng.choice([0.0, 1.5, 1e7, 3.25, -0.0], n, p=[0.4, 0.1, 0.2, 0.2, 0.1])
    if kind == "one":
        return np.full(n, 7.0)
    if kind == "mixed":     # half quiet years, a third at a limit, the rest distinct and of both signs
        x = rng.normal(0, 1e6, n)
        x[rng.random(n) < 0.5] = 0.0
        x[rng.random(n) < 0.33] = 2.5e6
        return x
    if kind == "special":
        x = rng.normal(0, 1, n)
        x[:: max(1, n // 9)] = np.inf
        x[1:: max(1, n // 7)] = -np.inf
        x.view(np.uint64)[n // 2:: max(1, n // 5)] = np.uint64(0xFFFFFFFFFFFFFFFF)   # the last in the order
        return x
    if kind == "sorted":
        return np.arange(n, dtype=np.float64)
    # "missed": the places the sample reads (j-th of S stretches, a fixed hash within it) hold one value
    b = 128
    while b < 1024 and b * 256 < n:
        b *= 2
    s = 4 * b
    x = rng.normal(0, 1e6, n)
    if n > 1024:
        j = np.arange(s, dtype=np.int64)
        a, e = j * n // s, (j + 1) * n // s
        x[a + ((((j * 2654435761) & 0xFFFFFFFF) * (e - a)) >> 32)] = -1e300
    return x


@pytest.mark.parametrize("kind", ["distinct", "few", "one", "mixed", "special", "sorted", "missed"])
@pytest.mark.parametrize("n", [1, 2, 3, 64, 65, 255, 256, 257, 513, 1023, 1024, 1025, 2049, 32768, 32769, 100_003, (1 << 18) + 1, 1 << 20,
                               (1 << 20) + 1])
def test_sort_desc(ara_lib, gpu_ctx, n, kind):
    import torch
    A = ara_lib
    if kind == "missed" and n > 300_000:
        pytest.skip("one workgroup sorts the whole bucket: kept to the smaller sizes")
    print(f"sort n={n} {kind}", flush=True)
    x = _values(kind, n, np.random.default_rng(n))
    want = _sorted(x)
    d = torch.from_numpy(x).cuda()
    out = torch.full((n,), 3.0, dtype=torch.float64, device="cuda")
    A.ara_sort_desc(gpu_ctx, d, out)
    A.ara_sync(gpu_ctx)
    assert out.cpu().numpy().tobytes() == want.tobytes()
    A.ara_sort_desc(gpu_ctx, d, d)      # in place
    A.ara_sync(gpu_ctx)
    assert d.cpu().numpy().tobytes() == want.tobytes()
