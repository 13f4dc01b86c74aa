"""The LDS-filter kernel at trial lengths around its chunks of 256 occurrences and segments of 1024, from every
position in a 16-byte group, with packed and 4-byte IDs and layers that few or nearly all events are in (the queue's
overflow), against the oracle.  Bound: two orders of the same non-negative terms, 1e-12 * max(|y|, P)."""
import math

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 2, 3, 4, 252, 253, 254, 255, 256, 257, 258, 508, 509, 510, 511, 512, 513, 514, 767, 768, 769, 1020, 1021,
         1022, 1023, 1024, 1025, 1026, 1279, 1280, 1281, 1535, 1537, 2047, 2048, 2049, 3001]


@pytest.mark.parametrize("packing", [0, 1])
@pytest.mark.parametrize("share", [0.02, 0.3, 0.97])
@pytest.mark.parametrize("start", [0, 1, 2, 3])
def test_chunks_against_oracle(ara_lib, gpu_ctx, packing, share, start):
    import torch
    from paper_1308_2066_amd import session
    A = ara_lib
    print(f"filter chunks packing={packing} share={share} start={start}", flush=True)
    rng = np.random.default_rng(17 + start)
    catalog, order = 30_000, rng.permutation(EDGES)
    lengths = np.concatenate([[start], order, rng.integers(0, 600, 40), order])
    offs = np.zeros(len(lengths) + 1, np.int64)
    np.cumsum(lengths, out=offs[1:])
    n = len(lengths)
    ids = rng.integers(0, catalog, size=int(offs[-1])).astype(np.int32)
    elts = [synth.elt_sparse(rng, int(share * catalog), catalog, 10.0, 2.0)]
    w = synth.Workload("filter", ids, offs, catalog, elts, (0.0, math.inf, 1e4, 1e9), None, (10.0,), 0)
    A.ara_set_option(gpu_ctx, A.ARA_OPT_YET_PACKING, packing)
    A.ara_set_option(gpu_ctx, A.ARA_OPT_PLACEMENT, A.ARA_PLACE_LDS_BITMAP)
    try:
        an = session.open_analysis(gpu_ctx, ids, offs, catalog, elts, w.layer_terms)
        try:
            y = torch.empty(n, dtype=torch.float64, device="cuda")
            A.ara_analyze(gpu_ctx, an.yet, an.layer, 0, n, y)
            A.ara_sync(gpu_ctx)
            y = y.cpu().numpy()
            ref = oracle.analyze_workload(w)
            assert np.all(np.abs(y - ref["ylt"]) <= 1e-12 * np.maximum(np.abs(ref["ylt"]), ref["occ_total"]))
            part = torch.empty(n - 7, dtype=torch.float64, device="cuda")
            A.ara_analyze(gpu_ctx, an.yet, an.layer, 5, n - 2, part)
            A.ara_sync(gpu_ctx)
            assert part.cpu().numpy().tobytes() == y[5:n - 2].tobytes()
        finally:
            an.release()
    finally:
        A.ara_set_option(gpu_ctx, A.ARA_OPT_YET_PACKING, 1)
        A.ara_set_option(gpu_ctx, A.ARA_OPT_PLACEMENT, A.ARA_PLACE_AUTO)


@pytest.mark.parametrize("catalog", [(1 << 20) - 1, 1 << 20, (1 << 20) + 1, 1_310_000, 2_500_000, 9_000_001])
@pytest.mark.parametrize("packing", [0, 1])
def test_folded_filter(ara_lib, gpu_ctx, catalog, packing):
    """Catalogs around and past the filter's 2^20 bits, half of the occurrences of events that share their bit with one
    in the layer but are not in it; the largest occurrences are exact and a batch gives the same bits."""
    import torch
    from paper_1308_2066_amd import session
    A = ara_lib
    print(f"folded filter catalog={catalog} packing={packing}", flush=True)
    rng = np.random.default_rng(catalog)
    n = 700
    lengths = rng.integers(0, 320, n)
    offs = np.zeros(n + 1, np.int64)
    np.cumsum(lengths, out=offs[1:])
    elts = [synth.elt_sparse(rng, 8_000, catalog, 10.0, 2.0) for _ in range(3)]
    inside = np.concatenate([e[0] for e in elts])
    ids = rng.integers(0, catalog, size=int(offs[-1]))
    near = rng.random(len(ids)) < 0.7
    ids[near] = (rng.choice(inside, int(near.sum())) % (1 << 20)) + (1 << 20) * rng.integers(
        0, max(1, -(-catalog // (1 << 20))), int(near.sum()))
    ids = np.minimum(ids, catalog - 1).astype(np.int32)
    w = synth.Workload("folded", ids, offs, catalog, elts, (0.0, math.inf, 1e4, 1e9), None, (10.0,), 0)
    A.ara_set_option(gpu_ctx, A.ARA_OPT_YET_PACKING, packing)
    try:
        an = session.open_analysis(gpu_ctx, ids, offs, catalog, elts, w.layer_terms)
    finally:
        A.ara_set_option(gpu_ctx, A.ARA_OPT_YET_PACKING, 1)
    try:
        y, z = (torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(2))
        A.ara_analyze(gpu_ctx, an.yet, an.layer, 0, n, y)
        A.ara_sync(gpu_ctx)
        ref = oracle.analyze_workload(w)
        tol = 1e-12 * np.maximum(np.abs(ref["ylt"]), ref["occ_total"])
        assert np.all(np.abs(y.cpu().numpy() - ref["ylt"]) <= tol)
        for t0, t1 in ((0, n), (13, n - 5), (3, 4)):
            A.ara_analyze_occ_max(gpu_ctx, an.yet, an.layer, t0, t1, z[t0:t1])
            A.ara_sync(gpu_ctx)
            assert z[t0:t1].cpu().numpy().tobytes() == ref["occ_max"][t0:t1].tobytes()
        batch = A.ara_batch_create(gpu_ctx, [(an.yet, an.layer, 0, n, z)])
        A.ara_batch_run(batch)
        A.ara_sync(gpu_ctx)
        assert z.cpu().numpy().tobytes() == y.cpu().numpy().tobytes()
        A.ara_batch_release(batch)
        A.ara_set_option(gpu_ctx, A.ARA_OPT_PLACEMENT, A.ARA_PLACE_GLOBAL_DENSE)
        A.ara_analyze(gpu_ctx, an.yet, an.layer, 0, n, z)
        A.ara_sync(gpu_ctx)
        assert np.all(np.abs(z.cpu().numpy() - ref["ylt"]) <= tol)
    finally:
        A.ara_set_option(gpu_ctx, A.ARA_OPT_PLACEMENT, A.ARA_PLACE_AUTO)
        an.release()
