"""Lane-per-trial kernels at the edges of their ID windows, tables and staging (IDs staged through LDS or read by the
lane, packed or int32): the oracle's sequential sums bit for bit, plain and batched, whole and on sub-ranges."""
import math

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("catalog", [1, 2, 1000, 12_268, 12_269, 12_270, 12_287, 12_288, 20_480])
@pytest.mark.parametrize("n,kind", [(1, "one"), (63, "edges"), (64, "edges"), (700, "edges"), (3000, "poisson")])
def test_lane_bits(ara_lib, gpu_ctx, catalog, n, kind):
    import torch
    from paper_1308_2066_amd import session
    A = ara_lib
    print(f"lane catalog={catalog} n={n} {kind}", flush=True)
    rng = np.random.default_rng(catalog + n)
    if kind == "poisson":
        lens = rng.poisson(100.0, size=n)
    else:      # window and group edges, empty trials, one much longer
        lens = np.array([0, 1, 3, 4, 5, 15, 16, 17, 31, 32, 33, 63, 64, 65, 0, 97, 128, 131])[np.arange(n) % 18]
        lens[n // 2] = 5000 + n
    offs = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=offs[1:])
    ids = rng.integers(0, catalog, size=int(offs[-1])).astype(np.int32)
    elts = [synth.elt_sparse(rng, max(1, catalog // 2), catalog, 10.0, 2.0) for _ in range(3)]
    w = synth.Workload("lane", ids, offs, catalog, elts, (5e3, 1e6, 1e5, math.inf), None, (10.0,), 0)
    ref = oracle.analyze_workload(w)["ylt"]
    A.ara_set_option(gpu_ctx, A.ARA_OPT_TRIAL_MODE, 2)
    try:
        for packing in (1, 0):
            A.ara_set_option(gpu_ctx, A.ARA_OPT_YET_PACKING, packing)
            an = session.open_analysis(gpu_ctx, ids, offs, catalog, elts, w.layer_terms)
            try:
                for block in (0, 512, 1024):
                    A.ara_set_option(gpu_ctx, A.ARA_OPT_BLOCK_THREADS, block)
                    for t0, t1 in {(0, n), (n // 3, n), (0, max(1, n - 1)), (n // 2, n // 2 + 1)}:
                        y = torch.full((t1 - t0,), math.nan, dtype=torch.float64, device="cuda")
                        A.ara_analyze(gpu_ctx, an.yet, an.layer, t0, t1, y)
                        A.ara_sync(gpu_ctx)
                        assert y.cpu().numpy().tobytes() == ref[t0:t1].tobytes(), (packing, block, t0, t1)
                A.ara_set_option(gpu_ctx, A.ARA_OPT_BLOCK_THREADS, 0)
                ys = [torch.full((n,), math.nan, dtype=torch.float64, device="cuda") for _ in range(2)]
                batch = A.ara_batch_create(gpu_ctx, [(an.yet, an.layer, 0, n, y) for y in ys])
                A.ara_batch_run(batch)
                A.ara_batch_run(batch)
                A.ara_sync(gpu_ctx)
                A.ara_batch_release(batch)
                assert all(y.cpu().numpy().tobytes() == ref.tobytes() for y in ys), packing
            finally:
                A.ara_set_option(gpu_ctx, A.ARA_OPT_BLOCK_THREADS, 0)
                an.release()
    finally:
        A.ara_set_option(gpu_ctx, A.ARA_OPT_TRIAL_MODE, 0)
        A.ara_set_option(gpu_ctx, A.ARA_OPT_YET_PACKING, 1)


@pytest.mark.parametrize("catalog,bad", [(1000, 1000), (1000, 70_000), (12_288, 12_288), (1000, -1)])
def test_lane_reports_ids_changed_out_of_range(ara_lib, gpu_ctx, catalog, bad):
    """An ID of a borrowed array changed after the YET was created: reported by the trial's
    own range only (int32 form)."""
    import torch
    A = ara_lib
    A.ara_set_option(gpu_ctx, A.ARA_OPT_YET_PACKING, 0)
    try:
        ids = torch.zeros(400, dtype=torch.int32, device="cuda")
        offs = torch.arange(0, 401, 50, dtype=torch.int64, device="cuda")
        yet = A.ara_yet_create(gpu_ctx, ids, offs, catalog)
        elt = A.ara_elt_create(gpu_ctx, torch.zeros(1, dtype=torch.int32, device="cuda"),
                               torch.ones(1, dtype=torch.float64, device="cuda"), catalog)
        layer = A.ara_layer_create(gpu_ctx, [elt], catalog, (0.0, math.inf, 0.0, math.inf))
        y = torch.empty(8, dtype=torch.float64, device="cuda")
        ids[133] = bad                                  # trial 2
        A.ara_analyze(gpu_ctx, yet, layer, 3, 8, y[:5])
        A.ara_sync(gpu_ctx)                              # not in range: no error
        A.ara_analyze(gpu_ctx, yet, layer, 0, 2, y[:2])
        A.ara_sync(gpu_ctx)
        A.ara_analyze(gpu_ctx, yet, layer, 0, 8, y)
        with pytest.raises(A.AraError) as e:
            A.ara_sync(gpu_ctx)
        assert e.value.status == A.ARA_E_EVENT_ID_RANGE
        A.ara_layer_release(layer)
        A.ara_elt_release(elt)
        A.ara_yet_release(yet)
    finally:
        A.ara_set_option(gpu_ctx, A.ARA_OPT_YET_PACKING, 1)
