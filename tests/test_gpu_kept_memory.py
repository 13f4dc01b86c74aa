"""Device memory that released handles leave with their context: reused by handles of nearly the same size with the same
results, bounded, and given back when the context is destroyed."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_reused_and_given_back(ara_lib):
    import torch
    from paper_1308_2066_amd import session
    A = ara_lib
    side = torch.cuda.Stream()
    ctx = A.ara_ctx_create(0)
    try:
        for k, n in enumerate((3000, 3010, 2500, 3000)):
            rng = np.random.default_rng(k)
            C = 40_000
            ids, offs = synth.yet_poisson(rng, n, 300.0, C)
            elts = [synth.elt_sparse(rng, 9_000, C, 10.0, 2.0) for _ in range(3)]
            w = synth.Workload("kept", ids, offs, C, elts, (5e4, 1e6, 2e5, 5e7), None, (10.0,), 0)
            A.ara_ctx_set_stream(ctx, side if k % 2 else None)
            an = session.open_analysis(ctx, ids, offs, C, elts, w.layer_terms)
            y = torch.empty(n, dtype=torch.float64, device="cuda")
            torch.cuda.synchronize()
            A.ara_analyze(ctx, an.yet, an.layer, 0, n, y)
            A.ara_sync(ctx)
            got = y.cpu().numpy()
            an.release()
            ref = oracle.analyze_workload(w)
            assert np.all(np.abs(got - ref["ylt"]) <= 1e-12 * np.maximum(np.abs(ref["ylt"]), ref["occ_total"])), k
    finally:
        A.ara_ctx_set_stream(ctx, None)
        A.ara_ctx_destroy(ctx)


def test_bounded(ara_lib):
    """Handles of 9 GiB in all leave at most 4 GiB with the context, none once it is gone."""
    import torch
    A = ara_lib
    ctx = A.ara_ctx_create(0)
    ids = torch.zeros(1, dtype=torch.int32, device="cuda")
    loss = torch.ones(1, dtype=torch.float64, device="cuda")
    slack = 256 << 20
    before = _free()
    elts = [A.ara_elt_create(ctx, ids, loss, 3 * (1 << 26) + k) for k in range(6)]       # 1.5 GiB tables
    assert before - _free() > 9 * (1 << 30)
    for e in elts:
        A.ara_elt_release(e)
    assert before - _free() <= (4 << 30) + slack
    A.ara_ctx_destroy(ctx)
    assert before - _free() <= slack
