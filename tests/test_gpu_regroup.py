"""The catalog-binned copy of a YET at the sizes where its build changes path: numbers of bins around the bits of a bin
number and the block tables' 64, trial lengths around a step (64), four steps, a chunk (1024) and past the staging LDS,
YETs around a counting block of 64 trials.  Checked through the tiled kernel: the largest occurrence is exact, the
YLT within 1e-12 * max(|y|, P), as two orders of the same non-negative terms."""
import math

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 63, 64, 65, 255, 256, 257, 511, 513, 1023, 1024, 1025, 2047, 2048, 2049, 5000]


@pytest.mark.parametrize("bins", [2, 4, 5, 8, 9, 16, 17, 32, 33, 63, 64, 65, 128, 129, 257])
@pytest.mark.parametrize("n,long_trials", [(64, False), (129, False), (300, True)])
def test_regrouped_against_oracle(ara_lib, gpu_ctx, bins, n, long_trials):
    from paper_1308_2066_amd import session
    import torch
    A = ara_lib
    print(f"regroup bins={bins} n={n} long={long_trials}", flush=True)
    rng = np.random.default_rng(bins * 1000 + n)
    catalog = (bins - 1) * 16384 + 5000
    lengths = np.resize(EDGES, n) + 8 * bins
    lengths[: len(EDGES)] = EDGES                     # and the edges themselves
    if long_trials:
        lengths[n // 2] = 40_000                      # a block past the staging LDS
    offs = np.zeros(n + 1, np.int64)
    np.cumsum(lengths, out=offs[1:])
    ids = rng.integers(0, catalog, size=int(offs[-1])).astype(np.int32)
    skew = rng.random(len(ids)) < 0.3                 # a bin that most lanes of a step share
    ids[skew] = rng.integers(0, 16384, size=int(skew.sum()))
    elts = [synth.elt_sparse(rng, catalog // 3, catalog, 10.0, 2.0) for _ in range(2)]
    w = synth.Workload("regroup", ids, offs, catalog, elts, (5e4, math.inf, 0.0, math.inf), None, (10.0,), 0)
    an = session.open_analysis(gpu_ctx, ids, offs, catalog, elts, w.layer_terms)
    try:
        assert A.ara_yet_info(an.yet)[2] == 2, "no binned copy"
        ref = oracle.analyze_workload(w)
        y = torch.empty(n, dtype=torch.float64, device="cuda")
        A.ara_analyze(gpu_ctx, an.yet, an.layer, 0, n, y)
        A.ara_sync(gpu_ctx)
        tol = 1e-12 * np.maximum(np.abs(ref["ylt"]), ref["occ_total"])
        assert np.all(np.abs(y.cpu().numpy() - ref["ylt"]) <= tol)
        A.ara_analyze_occ_max(gpu_ctx, an.yet, an.layer, 0, n, y)
        A.ara_sync(gpu_ctx)
        assert y.cpu().numpy().tobytes() == ref["occ_max"].tobytes()
    finally:
        an.release()
