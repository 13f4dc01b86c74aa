"""Per-occurrence outputs at trial lengths around 128 and 1024 events from every place in a 16-event line, catalogs whose
bits fit in LDS and larger ones (folded bits), each subset of the outputs, against the oracle.  Gross and
occurrence-net losses are exact; cumulative and ceded ones are sums of at most a few thousand non-negative terms, bounded
by 1e-12 * max(1, P) with P the trial's total."""
import math

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 2, 15, 16, 17, 126, 127, 128, 129, 130, 255, 256, 257, 1007, 1008, 1009, 1022, 1023, 1024, 1025, 1039, 1040,
         2047, 2048, 2049, 3333]


@pytest.mark.parametrize("catalog", [30_000, 1_310_000, 1_311_000, 3_000_001])
@pytest.mark.parametrize("f32", [False, True])
def test_event_outputs(ara_lib, gpu_ctx, catalog, f32):
    import torch
    from paper_1308_2066_amd import session
    A = ara_lib
    print(f"event outputs catalog={catalog} f32={f32}", flush=True)
    rng = np.random.default_rng(catalog)
    lengths = np.concatenate([rng.permutation(EDGES), rng.integers(0, 40, 30), rng.permutation(EDGES)])
    offs = np.zeros(len(lengths) + 1, np.int64)
    np.cumsum(lengths, out=offs[1:])
    n, m = len(lengths), int(offs[-1])
    elts = [synth.elt_sparse(rng, 9_000, catalog, 10.0, 2.0) for _ in range(2)]
    inside = np.concatenate([e[0] for e in elts])
    ids = rng.integers(0, catalog, size=m)
    near = rng.random(m) < 0.6
    ids[near] = (rng.choice(inside, int(near.sum())) % (1 << 20)) + (1 << 20) * rng.integers(0, 3, int(near.sum()))
    ids = np.where(ids < catalog, ids, rng.choice(inside, m)).astype(np.int32)
    w = synth.Workload("events", ids, offs, catalog, elts, (1e4, 1e6, 1e5, 1e8), None, (10.0,), 0)
    an = session.open_analysis(gpu_ctx, ids, offs, catalog, elts, w.layer_terms, None, 1 if f32 else 0)
    try:
        ref = oracle.analyze_workload(w, per_event=True, dat_f32=f32)
        gross, occ = ref["gross"], ref["occ"]
        if f32:   # the binary32 combined table, then the occurrence terms in binary64
            gross = gross.astype(np.float32).astype(np.float64)
            occ = np.minimum(np.maximum(gross - 1e4, 0.0), 1e6)
        cum = np.concatenate([np.cumsum(occ[offs[t]:offs[t + 1]]) for t in range(n)])
        agg = np.minimum(np.maximum(cum - 1e5, 0.0), 1e8)
        before = np.concatenate([[0.0], agg[:-1]])
        before[offs[:-1][lengths > 0]] = 0.0
        want = {"gross": gross, "occ": occ, "cum": cum, "ced": agg - before}
        for t0, t1 in ((0, n), (3, n - 2)):
            e0, e1 = int(offs[t0]), int(offs[t1])
            for names in (("gross", "occ", "cum", "ced"), ("cum",), ("gross", "ced"), ("occ",)):
                out = {k: torch.full((e1 - e0,), math.nan, dtype=torch.float64, device="cuda") for k in names}
                ylt = torch.full((t1 - t0,), math.nan, dtype=torch.float64, device="cuda")
                A.ara_analyze_events(gpu_ctx, an.yet, an.layer, t0, t1, ylt, out.get("gross"), out.get("occ"),
                                     out.get("cum"), out.get("ced"))
                A.ara_sync(gpu_ctx)
                for k in names:
                    got, exp = out[k].cpu().numpy(), want[k][e0:e1]
                    if k in ("gross", "occ"):
                        assert np.array_equal(got, exp), (k, t0)
                    else:
                        P = np.repeat([cum[offs[t + 1] - 1] if lengths[t] else 0.0 for t in range(t0, t1)],
                                      lengths[t0:t1])
                        assert np.all(np.abs(got - exp) <= 1e-12 * np.maximum(1.0, P)), (k, t0)
                exp = np.asarray([agg[offs[t + 1] - 1] if lengths[t] else 0.0 for t in range(t0, t1)])
                P = np.asarray([cum[offs[t + 1] - 1] if lengths[t] else 0.0 for t in range(t0, t1)])
                assert np.all(np.abs(ylt.cpu().numpy() - exp) <= 1e-12 * np.maximum(1.0, P))
    finally:
        an.release()
