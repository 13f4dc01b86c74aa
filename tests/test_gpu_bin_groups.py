"""Tiled launches split over bin groups (few trials, many catalog bins) against the oracle, and whole launches of the
same YET (under capture, in a batch of many passes, on more streams than keep a workspace) against split ones, bit for
bit.  The bound is the tiled kernel's: two orders of the same non-negative terms, 1e-12 * max(|y|, P)."""
import math

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _open(A, ctx, n, bins, run_bytes=4, seed=3):
    from paper_1308_2066_amd import session
    rng = np.random.default_rng(seed + n + bins)
    catalog = (bins - 1) * 16384 + (1 if bins > 2 else 4200)      # the last bin nearly empty
    lengths = rng.poisson(8.2 * bins + 20, size=n)
    lengths[:: max(1, n // 7)] = 0                                # empty trials
    lengths[-1] = 40 * bins + 300                                 # runs of more than 32
    offs = np.zeros(n + 1, np.int64)
    np.cumsum(lengths, out=offs[1:])
    ids = rng.integers(0, catalog, size=int(offs[-1])).astype(np.int32)
    elts = [synth.elt_sparse(rng, catalog // 3, catalog, 10.0, 2.0) for _ in range(3)]
    w = synth.Workload("groups", ids, offs, catalog, elts, (5e4, 1e6, 1e5 * bins, math.inf), None, (10.0,), 0)
    A.ara_set_option(ctx, A.ARA_OPT_YET_RUN_BYTES, run_bytes)
    try:
        an = session.open_analysis(ctx, ids, offs, catalog, elts, w.layer_terms)
    finally:
        A.ara_set_option(ctx, A.ARA_OPT_YET_RUN_BYTES, 4)
    assert A.ara_yet_info(an.yet)[2] == 2, "no binned copy"
    return w, an


def _ylt(A, ctx, an, t0, t1, fn="ara_analyze"):
    import torch
    y = torch.full((t1 - t0,), math.nan, dtype=torch.float64, device="cuda")
    getattr(A, fn)(ctx, an.yet, an.layer, t0, t1, y)
    A.ara_sync(ctx)
    return y.cpu().numpy()


@pytest.mark.parametrize("n,bins,run_bytes", [(1, 2, 4), (65, 3, 4), (3000, 4, 3), (4032, 19, 4), (4033, 62, 4),
                                              (8065, 7, 3), (500, 130, 4)])
def test_split_against_oracle(ara_lib, gpu_ctx, n, bins, run_bytes):
    A = ara_lib
    print(f"bin groups n={n} bins={bins} run bytes {run_bytes}", flush=True)
    w, an = _open(A, gpu_ctx, n, bins, run_bytes)
    try:
        ref = oracle.analyze_workload(w)
        y = _ylt(A, gpu_ctx, an, 0, n)
        tol = 1e-12 * np.maximum(np.abs(ref["ylt"]), ref["occ_total"])
        assert np.all(np.abs(y - ref["ylt"]) <= tol)
        assert _ylt(A, gpu_ctx, an, 0, n, "ara_analyze_occ_max").tobytes() == ref["occ_max"].tobytes()
        for t0, t1 in {(0, 1), (n // 3, n // 3 + 1), (n // 2, n), (0, max(1, n - 1))}:
            if t1 <= n:
                assert _ylt(A, gpu_ctx, an, t0, t1).tobytes() == y[t0:t1].tobytes(), (t0, t1)
    finally:
        an.release()


def test_whole_launches_give_the_same_bits(ara_lib, gpu_ctx):
    import torch
    A = ara_lib
    n = 6000
    w, an = _open(A, gpu_ctx, n, 31)
    streams = [torch.cuda.Stream() for _ in range(6)]      # more than keep a workspace
    try:
        want = _ylt(A, gpu_ctx, an, 0, n)
        outs = [torch.full((n,), math.nan, dtype=torch.float64, device="cuda") for _ in streams]
        torch.cuda.synchronize()
        for s, o in zip(streams, outs):                     # overlapping launches, none waited for
            A.ara_ctx_set_stream(gpu_ctx, s)
            A.ara_analyze(gpu_ctx, an.yet, an.layer, 0, n, o)
        torch.cuda.synchronize()
        for o in outs:
            assert o.cpu().numpy().tobytes() == want.tobytes()
        # captured: replayed with the stream's own eager launches between the replays
        o, p = outs[0], outs[1]
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=streams[0]):
            A.ara_ctx_set_stream(gpu_ctx, torch.cuda.current_stream())
            A.ara_analyze(gpu_ctx, an.yet, an.layer, 0, n, o)
        for _ in range(3):
            o.fill_(math.nan)
            p.fill_(math.nan)
            torch.cuda.synchronize()
            graph.replay()
            A.ara_ctx_set_stream(gpu_ctx, streams[0])
            A.ara_analyze(gpu_ctx, an.yet, an.layer, 0, n, p)
            torch.cuda.synchronize()
            assert o.cpu().numpy().tobytes() == want.tobytes() and p.cpu().numpy().tobytes() == want.tobytes()
    finally:
        A.ara_ctx_set_stream(gpu_ctx, torch.cuda.current_stream())
        an.release()


@pytest.mark.parametrize("copies", [1, 600])
def test_batch_split_and_whole(ara_lib, gpu_ctx, copies):
    """A batch of few passes is split over bin groups, one of many passes is not."""
    import torch
    A = ara_lib
    n = 5000
    w, an = _open(A, gpu_ctx, n, 12)
    ylts = [torch.full((n,), math.nan, dtype=torch.float64, device="cuda") for _ in range(copies)]
    batch = A.ara_batch_create(gpu_ctx, [(an.yet, an.layer, 0, n, y) for y in ylts])
    try:
        want = _ylt(A, gpu_ctx, an, 0, n)
        for _ in range(2):
            for y in ylts:
                y.fill_(math.nan)
            A.ara_batch_run(batch)
            A.ara_sync(gpu_ctx)
            assert all(y.cpu().numpy().tobytes() == want.tobytes() for y in ylts)
    finally:
        A.ara_batch_release(batch)
        an.release()
