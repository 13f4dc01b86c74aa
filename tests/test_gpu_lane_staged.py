"""Plain launches of the lane-per-trial kernel that stages its IDs through LDS (at least 512 trials per CU): the
oracle's sequential sums bit for bit around the largest tables that leave the waves their rows, and bad IDs, which only
the clamp keeps inside the table, reported by plain launches and by batches."""
import math

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _many():
    import torch
    return 512 * torch.cuda.get_device_properties(0).multi_processor_count


# 12,269 and 18,413: the largest tables beside 16 and 4 waves' rows
@pytest.mark.parametrize("catalog,block", [(1, 0), (700, 0), (12_268, 0), (12_269, 0), (12_270, 0), (12_269, 1024),
                                           (18_412, 256), (18_413, 256), (18_414, 256), (15_000, 512)])
def test_plain_staged_bits(ara_lib, gpu_ctx, catalog, block):
    import torch
    from paper_1308_2066_amd import session
    A = ara_lib
    n = _many() + 37
    print(f"staged catalog={catalog} block={block} n={n}", flush=True)
    rng = np.random.default_rng(catalog + block)
    lens = np.array([0, 1, 3, 4, 5, 9, 16, 2, 31, 32, 33, 7, 63, 6, 64, 65])[rng.integers(0, 16, size=n)]
    lens[n // 2] = 700
    offs = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=offs[1:])
    ids = rng.integers(0, catalog, size=int(offs[-1])).astype(np.int32)
    elts = [synth.elt_sparse(rng, max(1, catalog // 2), catalog, 10.0, 2.0) for _ in range(2)]
    w = synth.Workload("staged", ids, offs, catalog, elts, (5e3, 1e6, 1e5, math.inf), None, (10.0,), 0)
    ref = oracle.analyze_workload(w)["ylt"]
    try:
        A.ara_set_option(gpu_ctx, A.ARA_OPT_BLOCK_THREADS, block)
        for packing in (1, 0):
            A.ara_set_option(gpu_ctx, A.ARA_OPT_YET_PACKING, packing)
            an = session.open_analysis(gpu_ctx, ids, offs, catalog, elts, w.layer_terms)
            try:
                for t0, t1 in ((0, n), (37, n), (5, n - 30)):
                    y = torch.full((t1 - t0,), math.nan, dtype=torch.float64, device="cuda")
                    A.ara_analyze(gpu_ctx, an.yet, an.layer, t0, t1, y)
                    A.ara_sync(gpu_ctx)
                    assert y.cpu().numpy().tobytes() == ref[t0:t1].tobytes(), (packing, t0, t1)
            finally:
                an.release()
    finally:
        A.ara_set_option(gpu_ctx, A.ARA_OPT_BLOCK_THREADS, 0)
        A.ara_set_option(gpu_ctx, A.ARA_OPT_YET_PACKING, 1)


@pytest.mark.parametrize("catalog,bad", [(1000, 1000), (1000, 70_000), (12_269, 12_269), (12_269, -1), (1000, 65_535),
                                         (1000, 65_536)])
@pytest.mark.parametrize("batched", [False, True])
def test_staged_reports_ids_changed_out_of_range(ara_lib, gpu_ctx, catalog, bad, batched):
    """int32 IDs of a borrowed array, one changed after the YET was created: at each place of a 64-byte row."""
    import torch
    A = ara_lib
    n = 3000 if batched else _many() + 5
    A.ara_set_option(gpu_ctx, A.ARA_OPT_YET_PACKING, 0)
    try:
        ids = torch.full((40 * n + 1,), catalog - 1, dtype=torch.int32, device="cuda")[: 40 * n]
        offs = torch.arange(0, 40 * n + 1, 40, dtype=torch.int64, device="cuda")
        yet = A.ara_yet_create(gpu_ctx, ids, offs, catalog)
        elt = A.ara_elt_create(gpu_ctx, torch.tensor([catalog - 1], dtype=torch.int32, device="cuda"),
                               torch.ones(1, dtype=torch.float64, device="cuda"), catalog)
        layer = A.ara_layer_create(gpu_ctx, [elt], catalog, (0.0, math.inf, 0.0, math.inf))
        y = torch.empty(n, dtype=torch.float64, device="cuda")
        batch = A.ara_batch_create(gpu_ctx, [(yet, layer, 0, n, y)]) if batched else None

        def analyse():
            if batched:
                A.ara_batch_run(batch)
            else:
                A.ara_analyze(gpu_ctx, yet, layer, 0, n, y)
            A.ara_sync(gpu_ctx)
        analyse()
        assert float(y.min()) == float(y.max()) == 40.0
        for at in (0, 7, 40 * 999 + 33, 40 * n - 1):
            print(f"staged bad id {bad} of {catalog} at {at}, batched={batched}", flush=True)
            ids[at] = bad
            with pytest.raises(A.AraError) as e:
                analyse()
            assert e.value.status == A.ARA_E_EVENT_ID_RANGE
            ids[at] = catalog - 1
        analyse()
        if batch is not None:
            A.ara_batch_release(batch)
        A.ara_layer_release(layer)
        A.ara_elt_release(elt)
        A.ara_yet_release(yet)
    finally:
        A.ara_set_option(gpu_ctx, A.ARA_OPT_YET_PACKING, 1)
