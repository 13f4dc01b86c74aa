"""The server over a YET with a binned copy: requests of few and many trials give the same analysis' bits alone, nothing
is allocated while it serves, and its memory stays within the budget."""
import math

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
SLACK = 160 << 20


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("budget", [64 << 20, 1 << 30])
def test_tiled_requests(ara_lib, budget):
    """budget 64 MB: no room for the lanes' split workspaces (launches run whole)."""
    import torch
    from paper_1308_2066_amd import session
    A = ara_lib
    ctx = A.ara_ctx_create(0)
    rng = np.random.default_rng(31)
    bins, n = 24, 300_000
    catalog = bins * 16384 - 77
    lens = rng.integers(8 * bins + 4, 8 * bins + 40, size=n)
    offs = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=offs[1:])
    ids = rng.integers(0, catalog, size=int(offs[-1])).astype(np.int32)
    yet = A.ara_yet_create(ctx, session.to_device(ids), session.to_device(offs), catalog)
    assert A.ara_yet_info(yet)[2] == 2, "no binned copy"
    pool = []
    for _ in range(4):
        e, v = synth.elt_sparse(rng, 9_000, catalog, 10.0, 2.0)
        pool.append(A.ara_elt_create(ctx, session.to_device(e), session.to_device(v), catalog))
    rps = [2.0, 10.0, 100.0]
    before = _free()
    srv = A.ara_server_create(ctx, yet, pool, rps, max_batch=2, memory_budget=budget)
    try:
        assert before - _free() <= budget + SLACK
        asked = []
        for k in range(14):
            t0 = int(rng.integers(0, n // 2))
            t1 = (t0 + 60, t0 + 2500, n, n - 1)[k % 4]
            asked.append(([k % 4, (k + 1) % 4], (1e4, 1e6, 1e5, math.inf), t0, t1))
        held = _free()
        tickets = [A.ara_server_submit(srv, *r) for r in asked]
        got = [A.ara_server_wait(srv, t)[:2] for t in tickets]
        assert abs(_free() - held) <= 12 << 20          # the runtime takes 4 MB with the first launches
        for (idx, terms, t0, t1), (pml, tvar) in zip(asked, got):
            layer = A.ara_layer_create(ctx, [pool[i] for i in idx], catalog, terms)
            y = torch.empty(t1 - t0, dtype=torch.float64, device="cuda")
            A.ara_analyze(ctx, yet, layer, t0, t1, y)
            p, t = A.ara_risk_measures(ctx, y, rps)
            A.ara_layer_release(layer)
            assert p.tobytes() == pml.tobytes() and t.tobytes() == tvar.tobytes(), (t0, t1)
    finally:
        A.ara_server_release(srv)
        for e in pool:
            A.ara_elt_release(e)
        A.ara_yet_release(yet)
        A.ara_ctx_destroy(ctx)
