"""A saved schedule whose batch shape is longer than any line buffer is loaded back."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_long_batch_shape_round_trip(ara_lib, tmp_path):
    import torch
    from paper_1308_2066_amd import session
    A = ara_lib
    rng = np.random.default_rng(4)
    C, n, jobs = 3_000, 200, 1500
    ids, offs = synth.yet_poisson(rng, n, 20.0, C)
    elts = [synth.elt_sparse(rng, 800, C, 10.0, 2.0)]
    path, seen = str(tmp_path / "schedules.txt"), []
    for rep in range(2):
        ctx = A.ara_ctx_create(0)
        an = session.open_analysis(ctx, ids, offs, C, elts, (1e3, 1e6, 1e4, 2e6))
        out = torch.empty((jobs, n), dtype=torch.float64, device="cuda")
        if rep:
            A.ara_tune_cache_load(ctx, path)
        batch = A.ara_batch_create(ctx, [(an.yet, an.layer, 0, n, out[j]) for j in range(jobs)])
        A.ara_batch_run(batch)
        A.ara_sync(ctx)
        seen.append(A.ara_batch_info(batch))
        if not rep:
            A.ara_tune_cache_save(ctx, path)
        A.ara_batch_release(batch)
        an.release()
        A.ara_ctx_destroy(ctx)
    assert max(map(len, open(path))) > 8192
    assert seen[0] == seen[1]
