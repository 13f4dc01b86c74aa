"""A trial's year loss and largest occurrence do not depend on the other trials of its YET: shards of a YET, each a
handle of its own, give the whole YET's bits, however each launch is split over bins and workgroups."""
import math

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bins,n,run_bytes", [(2, 9000, 4), (19, 40_000, 4), (20, 9000, 3), (21, 60_000, 4),
                                              (62, 20_000, 4), (123, 20_000, 3)])
def test_shards_give_the_whole_yets_bits(ara_lib, gpu_ctx, bins, n, run_bytes):
    import torch
    from paper_1308_2066_amd import session
    A = ara_lib
    rng = np.random.default_rng(bins)
    catalog = (bins - 1) * 16384 + 5000
    lens = rng.poisson(8.1 * bins + 30, size=n)
    offs = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=offs[1:])
    ids = rng.integers(0, catalog, size=int(offs[-1])).astype(np.int32)
    elts = [synth.elt_sparse(rng, catalog // 3, catalog, 10.0, 2.0) for _ in range(2)]
    w = synth.Workload("shards", ids, offs, catalog, elts, (5e4, 1e6, 1e5 * bins, math.inf), None, (10.0,), 0)
    ref = oracle.analyze_workload(w)
    A.ara_set_option(gpu_ctx, A.ARA_OPT_YET_RUN_BYTES, run_bytes)
    an = session.open_analysis(gpu_ctx, ids, offs, catalog, elts, w.layer_terms)
    try:
        assert A.ara_yet_info(an.yet)[2] == 2, "no binned copy"
        y, m = (torch.full((n,), math.nan, dtype=torch.float64, device="cuda") for _ in range(2))
        A.ara_analyze(gpu_ctx, an.yet, an.layer, 0, n, y)
        A.ara_analyze_occ_max(gpu_ctx, an.yet, an.layer, 0, n, m)
        A.ara_sync(gpu_ctx)
        y, m = y.cpu().numpy(), m.cpu().numpy()
        assert np.all(np.abs(y - ref["ylt"]) <= 1e-12 * np.maximum(np.abs(ref["ylt"]), ref["occ_total"]))
        for t0, t1 in ((0, 1), (1, 70), (70, 1200), (1200, 5300), (5300, n)):
            print(f"shard of {bins} bins: trials {t0}-{t1}", flush=True)
            shard = A.ara_yet_create(gpu_ctx, session.to_device(ids[offs[t0]:offs[t1]]),
                                     session.to_device(offs[t0:t1 + 1] - offs[t0]), catalog)
            assert A.ara_yet_info(shard)[2] == 2, "no binned copy"
            ys, ms = (torch.full((t1 - t0,), math.nan, dtype=torch.float64, device="cuda") for _ in range(2))
            A.ara_analyze(gpu_ctx, shard, an.layer, 0, t1 - t0, ys)
            A.ara_analyze_occ_max(gpu_ctx, shard, an.layer, 0, t1 - t0, ms)
            A.ara_sync(gpu_ctx)
            A.ara_yet_release(shard)
            assert ys.cpu().numpy().tobytes() == y[t0:t1].tobytes(), (t0, t1)
            assert ms.cpu().numpy().tobytes() == m[t0:t1].tobytes(), (t0, t1)
    finally:
        A.ara_set_option(gpu_ctx, A.ARA_OPT_YET_RUN_BYTES, 4)
        an.release()
