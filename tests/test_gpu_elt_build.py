"""Direct access tables from an ELT's records at the edges of the build's stretches: catalogs of part of a word to several
128 KB stretches, no records to more than one launch takes, records in any order, rebuilt after they moved; and its
errors (an ID outside the catalog, a bad loss, an event twice, wherever they stand).  Lookups are exact."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _elt(A, ctx, ids, losses, catalog, precision=0):
    import torch
    i = torch.from_numpy(np.ascontiguousarray(ids, np.int32)).cuda()
    l = torch.from_numpy(np.ascontiguousarray(losses, np.float64)).cuda()
    return A.ara_elt_create(ctx, i, l, catalog, None, precision), i, l


def _gross(A, ctx, layer, catalog):
    import torch
    g = torch.full((catalog,), math.nan, dtype=torch.float64, device="cuda")
    A.ara_lookup(ctx, layer, torch.arange(catalog, dtype=torch.int32, device="cuda"), g, None)
    A.ara_sync(ctx)
    return g.cpu().numpy()


@pytest.mark.parametrize("catalog", [1, 31, 32, 33, 1000, 65_537, 1_048_576, 1_048_577, 2_500_000])
@pytest.mark.parametrize("n_elts,records", [(1, 0), (1, 1), (3, 1023), (1, 8193), (40, 500), (2, 200_000)])
def test_tables(ara_lib, gpu_ctx, catalog, n_elts, records):
    A = ara_lib
    print(f"elt build catalog={catalog} elts={n_elts} records={records}", flush=True)
    rng = np.random.default_rng(catalog + records)
    records = min(records, catalog)
    made, want = [], np.zeros(catalog)
    for k in range(n_elts):
        ids = rng.choice(catalog, size=records, replace=False)
        if records > 2:      # the ends of the catalog
            ids = np.unique(np.concatenate([ids, [0, catalog - 1]]))
            rng.shuffle(ids)
        losses = rng.integers(1, 1000, size=len(ids)).astype(np.float64)
        made.append(_elt(A, gpu_ctx, ids, losses, catalog) + (ids, losses))
        want[ids] += losses      # whole numbers: exact in any order
    layer = A.ara_layer_create(gpu_ctx, [m[0] for m in made], catalog, (0.0, math.inf, 0.0, math.inf))
    try:
        assert np.array_equal(_gross(A, gpu_ctx, layer, catalog), want)
        moved = np.zeros(catalog)
        for _, i, l, ids, losses in made:      # the records of other events, then rebuilt
            new = rng.permutation(catalog)[: len(ids)] if catalog < 100_000 else (ids + 12345) % catalog
            import torch
            i.copy_(torch.from_numpy(new.astype(np.int32)))
            moved[new] += losses
        A.ara_layer_build(gpu_ctx, layer, A.ARA_BUILD_TABLES)
        assert np.array_equal(_gross(A, gpu_ctx, layer, catalog), moved)
    finally:
        A.ara_layer_release(layer)
        for m in made:
            A.ara_elt_release(m[0])


@pytest.mark.parametrize("records", [5, 1024, 20_000, 140_000])
@pytest.mark.parametrize("where", [0, 1, -1])
def test_errors(ara_lib, gpu_ctx, records, where):
    A = ara_lib
    catalog = 1_500_000
    print(f"elt build errors records={records} where={where}", flush=True)
    rng = np.random.default_rng(records)
    ids = rng.choice(catalog, size=records, replace=False)
    losses = rng.uniform(1, 10, records)
    at = where % records
    for kind, code in (("range", A.ARA_E_EVENT_ID_RANGE), ("negative", A.ARA_E_EVENT_ID_RANGE), ("loss", A.ARA_E_BAD_LOSS),
                       ("nan", A.ARA_E_BAD_LOSS), ("twice", A.ARA_E_DUP_EVENT)):
        i, l = ids.copy(), losses.copy()
        if kind == "range":
            i[at] = catalog
        elif kind == "negative":
            i[at] = -1
        elif kind == "loss":
            l[at] = -1.0
        elif kind == "nan":
            l[at] = math.nan
        else:
            i[at] = i[at - 2]
        with pytest.raises(A.AraError) as e:
            _elt(A, gpu_ctx, i, l, catalog)
        assert e.value.status == code, kind
