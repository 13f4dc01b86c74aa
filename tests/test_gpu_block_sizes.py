"""Device memory taken for handles: what is too large to be kept is allocated as asked, and a server's arena stays within
its budget."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
SLACK = 160 << 20          # granularity of the mappings, pinned staging, the runtime's own


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_large_block_is_not_rounded(ara_lib):
    """A packed copy of just over 4.5 GiB."""
    import torch
    A = ara_lib
    ctx = A.ara_ctx_create(0)
    n = (9 * (1 << 29)) // 3 + 4096                                 # 3 bytes an event
    ids = torch.zeros(n, dtype=torch.int32, device="cuda")
    offs = torch.arange(0, n + 1, 4096, dtype=torch.int64, device="cuda")
    offs = torch.cat([offs, torch.tensor([n], device="cuda")]) if int(offs[-1]) != n else offs
    before = _free()
    yet = A.ara_yet_create(ctx, ids, offs, 10_000)
    try:
        assert A.ara_yet_info(yet)[2] == 3
        assert before - _free() <= 3 * n + SLACK
    finally:
        A.ara_yet_release(yet)
        A.ara_ctx_destroy(ctx)


def test_server_arena_within_its_budget(ara_lib):
    import torch
    from paper_1308_2066_amd import session
    A = ara_lib
    ctx = A.ara_ctx_create(0)
    rng = np.random.default_rng(2)
    C, n = 2_000, 1_000
    ids, offs = synth.yet_poisson(rng, n, 20.0, C)
    an = session.open_analysis(ctx, ids, offs, C, [synth.elt_sparse(rng, 500, C, 10.0, 2.0)], (0.0, 1e9, 0.0, 1e9))
    budget = (8 << 30) + (16 << 20)
    before = _free()
    srv = A.ara_server_create(ctx, an.yet, an.elts, [10.0], max_batch=2, memory_budget=budget)
    try:
        assert before - _free() <= budget + SLACK
    finally:
        A.ara_server_release(srv)
        an.release()
        A.ara_ctx_destroy(ctx)
