"""Risk measures by selection (k_risk.hip) at the sizes and distributions where it could go wrong, against the
oracle: PML is an order statistic (bit-exact), TVaR within the rounding bound of a k-term sum of one sign."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _ylt(n, kind):
    rng = np.random.default_rng(n * 11 + sum(map(ord, kind)))
    y = rng.lognormal(13, 2.2, size=n)
    if kind == "capped":        # quiet years, and more than a rank's worth at the limit
        y = np.minimum(y, np.quantile(y, 0.7))
        y[rng.random(n) < 0.25] = 0.0
    elif kind == "zeros":       # all but a few quiet
        y[rng.random(n) < 0.999] = 0.0
    elif kind == "all_zero":
        y[:] = 0.0
        y[::2] = -0.0
    elif kind == "below_zero":  # zeros in the middle of the order; all the k largest of one sign
        y = y - np.quantile(y, 0.2)
        y[rng.random(n) < 0.1] = 0.0
    elif kind == "close":       # half of the losses agree in more bits than two rounds of bins tell apart
        near = rng.random(n) < 0.5
        y[near] = float(np.quantile(y, 0.995)) * (1.0 + rng.integers(0, 1 << 14, size=int(near.sum())) * 2.0 ** -40)
    elif kind == "round":       # keys on the bins' edges
        y = rng.integers(0, 64, size=n) * 10.0
    elif kind == "inf":
        y[rng.random(n) < 0.02] = np.inf
    return y


SHORT = [(n, k) for n in (1, 2, 4, 5, 63, 64, 65, 2047, 2049, 10_000) for k in ("distinct", "capped", "round")]
KINDS = ("distinct", "capped", "zeros", "all_zero", "below_zero", "close", "round", "inf")


@pytest.mark.parametrize("n,kind", SHORT + [(n, k) for n in (16_384, 16_385, 131_073, 600_001) for k in KINDS])
def test_selection(ara_lib, gpu_ctx, n, kind):
    import torch
    A = ara_lib
    print(f"risk selection n={n} kind={kind}", flush=True)
    y = _ylt(n, kind)
    # 20 return periods: two groups of ranks; below_zero stays among the positive losses
    rps = [10.0, 100.0, 250.0, float(n)] + list(np.geomspace(2.0 if kind == "below_zero" else 1.0, max(2.0, n / 2.0), 16))
    pml_o, tvar_o, ranks, _ = oracle.risk(y, rps)
    yt = torch.from_numpy(y).cuda()
    pml, tvar = A.ara_risk_measures(gpu_ctx, yt, rps)
    assert np.asarray(pml).tobytes() == np.asarray(pml_o).tobytes()
    with np.errstate(invalid="ignore"):
        bound = 2.0 * np.asarray(ranks, float) * 2.0 ** -53 * np.abs(tvar_o) + 1e-300
        same = (tvar == tvar_o) | (np.abs(tvar - tvar_o) <= bound)
    assert same.all(), (tvar, tvar_o)
    if n <= A.ARA_NOALLOC_MAX_N:   # a workspace of another alignment, and again
        p2, t2 = A.ara_risk_measures_noalloc(gpu_ctx, yt, rps)
        ws = torch.empty(A.ara_sort_workspace_size(n) + 8, dtype=torch.uint8, device="cuda")[8:]
        p3, t3 = A.ara_risk_measures(gpu_ctx, yt, rps, ws)
        for p, t in ((p2, t2), (p3, t3)):
            assert p.tobytes() == pml.tobytes() and t.tobytes() == tvar.tobytes()


@pytest.mark.parametrize("share", [63, 64, 65, 700, 1023, 1024, 1025])
@pytest.mark.parametrize("n", [9_000, 100_000])
def test_shared_losses(ara_lib, gpu_ctx, n, share):
    """Every loss occurs `share` times, next to its neighbour in binary64 (so two or more losses fall in a bin), or
    alone in its bin."""
    import torch
    A = ara_lib
    rng = np.random.default_rng(share)
    print(f"shared losses n={n} share={share}", flush=True)
    v = np.repeat(rng.lognormal(13, 2.2, size=n // share + 1), share)[:n]
    near = rng.random(n) < 0.3
    v[near] = np.nextafter(v[near], np.inf)
    y = rng.permutation(v)
    rps = [10.0, 50.0, 250.0, 1000.0, float(n)]
    pml_o, tvar_o, ranks, _ = oracle.risk(y, rps)
    pml, tvar = A.ara_risk_measures(gpu_ctx, torch.from_numpy(y).cuda(), rps)
    assert np.asarray(pml).tobytes() == np.asarray(pml_o).tobytes()
    assert np.all(np.abs(tvar - tvar_o) <= 2.0 * np.asarray(ranks, float) * 2.0 ** -53 * np.abs(tvar_o) + 1e-300)


def test_batch_of_short_and_long(ara_lib, gpu_ctx):
    """A batch of YLTs on both sides of the one-workgroup limit, two sets of return periods:
    the same bits as one call per YLT."""
    import torch
    import synth
    from paper_1308_2066_amd import session
    A = ara_lib
    rng = np.random.default_rng(5)
    n, C = 40_000, 3_000
    ids, offs = synth.yet_poisson(rng, n, 12.0, C)
    an = session.open_analysis(gpu_ctx, ids, offs, C, [synth.elt_sparse(rng, 900, C, 10.0, 2.0)],
                               (1e3, 1e6, 1e4, 2e6))
    ranges = [(0, n), (5, 6), (100, 16_484), (100, 16_485), (0, 20_000), (39_000, n)]
    ylts = [torch.empty(b - a, dtype=torch.float64, device="cuda") for a, b in ranges]
    batch = A.ara_batch_create(gpu_ctx, [(an.yet, an.layer, a, b, y) for (a, b), y in zip(ranges, ylts)])
    try:
        A.ara_batch_run(batch)
        for rps in ([10.0, 100.0, 250.0], list(np.geomspace(1.0, 500.0, 19)), [10.0, 100.0, 250.0]):
            for _ in range(2):
                pml, tvar = A.ara_batch_risk(batch, rps)
                for j, y in enumerate(ylts):
                    p, t = A.ara_risk_measures(gpu_ctx, y, rps)
                    assert p.tobytes() == pml[j].tobytes() and t.tobytes() == tvar[j].tobytes(), (j, len(rps))
    finally:
        A.ara_batch_release(batch)
        an.release()


@pytest.mark.parametrize("few", (10.0, 40.0))
@pytest.mark.parametrize("n", (1_500, 10_000, 16_384, 16_385, 600_001))
def test_one_loss_but_for_a_few(ara_lib, gpu_ctx, n, few):
    """A sample of one value says nothing about the range: the few other losses, whose keys differ from it in the
    high bits alone, belong in the last bin (or below the bins)."""
    import torch
    A = ara_lib
    print(f"risk one loss n={n} few={few}", flush=True)
    y = np.full(n, 20.0)
    y[[n // 3, n // 2 + 1, n - 2]] = few
    rps = [1.0, 10.0, 100.0, float(n)]
    pml_o, tvar_o, ranks, _ = oracle.risk(y, rps)
    pml, tvar = A.ara_risk_measures(gpu_ctx, torch.from_numpy(y).cuda(), rps)
    assert np.asarray(pml).tobytes() == np.asarray(pml_o).tobytes()
    assert np.asarray(tvar).tobytes() == np.asarray(tvar_o).tobytes()   # sums of whole numbers below 2^53


@pytest.mark.parametrize("longest", (9, 18))
def test_batch_of_many_long(ara_lib, gpu_ctx, longest):
    """More long YLTs than the passes have workgroups for at 4096 losses each (in the collection; in both): the same
    bits as one call per YLT."""
    import torch
    import synth
    from paper_1308_2066_amd import session
    A = ara_lib
    rng = np.random.default_rng(6)
    n, C = 120_000, 3_000
    ids, offs = synth.yet_poisson(rng, n, 3.0, C)
    an = session.open_analysis(gpu_ctx, ids, offs, C, [synth.elt_sparse(rng, 900, C, 10.0, 2.0)],
                               (1e3, 1e6, 1e4, 2e6))
    ranges = [(j, n) for j in range(longest)] + [(0, 16_385), (7, 30_000)]
    ylts = [torch.empty(b - a, dtype=torch.float64, device="cuda") for a, b in ranges]
    batch = A.ara_batch_create(gpu_ctx, [(an.yet, an.layer, a, b, y) for (a, b), y in zip(ranges, ylts)])
    try:
        A.ara_batch_run(batch)
        for rps in ([10.0, 100.0, 250.0], list(np.geomspace(1.0, 500.0, 19))):
            pml, tvar = A.ara_batch_risk(batch, rps)
            for j, y in enumerate(ylts):
                p, t = A.ara_risk_measures(gpu_ctx, y, rps)
                assert p.tobytes() == pml[j].tobytes() and t.tobytes() == tvar[j].tobytes(), (j, len(rps))
    finally:
        A.ara_batch_release(batch)
        an.release()
