"""A batch whose split sums do not fit in device memory is created all the same, and gives the plain launches' bits."""
import math

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_batch_without_room_for_its_sums(ara_lib):
    import torch
    from paper_1308_2066_amd import session
    A = ara_lib
    ctx = A.ara_ctx_create(0)
    A.ara_set_option(ctx, A.ARA_OPT_KEPT_BYTES, 0)
    rng = np.random.default_rng(8)
    bins, n, copies = 20, 40_000, 100
    catalog = bins * 16384
    lens = rng.integers(8 * bins + 4, 8 * bins + 30, size=n)
    offs = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=offs[1:])
    ids = rng.integers(0, catalog, size=int(offs[-1])).astype(np.int32)
    an = session.open_analysis(ctx, ids, offs, catalog, [synth.elt_sparse(rng, catalog // 3, catalog, 10.0, 2.0)],
                               (5e4, 1e6, 1e5 * bins, math.inf))
    assert A.ara_yet_info(an.yet)[2] == 2, "no binned copy"
    want = torch.empty(n, dtype=torch.float64, device="cuda")
    A.ara_analyze(ctx, an.yet, an.layer, 0, n, want)
    ylts = [torch.full((n,), math.nan, dtype=torch.float64, device="cuda") for _ in range(copies)]
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    # all but 64 MB taken (what the device reports as free is less than what can be had); the sums take 250 MB
    hog = [torch.empty(torch.cuda.mem_get_info()[0] - (96 << 20), dtype=torch.uint8, device="cuda")]
    try:
        while True:
            hog.append(torch.empty(32 << 20, dtype=torch.uint8, device="cuda"))
    except torch.OutOfMemoryError:
        del hog[-2:]
    torch.cuda.empty_cache()
    batch = None
    try:
        batch = A.ara_batch_create(ctx, [(an.yet, an.layer, 0, n, y) for y in ylts])
        for _ in range(2):
            A.ara_batch_run(batch)
            A.ara_sync(ctx)
        bits = want.cpu().numpy().tobytes()
        assert all(y.cpu().numpy().tobytes() == bits for y in ylts)
    finally:
        if batch is not None:
            A.ara_batch_release(batch)
        del hog
        torch.cuda.empty_cache()
        an.release()
        A.ara_ctx_destroy(ctx)
