"""What a context keeps of released handles' device memory is reused, and goes back on request, when the context is
destroyed, and when another context on the device needs it."""
import pytest

pytestmark = pytest.mark.gpu
GIB = 1 << 30
SLACK = 64 << 20


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def _table(A, ctx, gib):
    """An ELT whose binary64 table takes gib GiB (and a 64th of it in seen bits)."""
    import torch
    ids = torch.zeros(1, dtype=torch.int32, device="cuda")
    loss = torch.ones(1, dtype=torch.float64, device="cuda")
    return A.ara_elt_create(ctx, ids, loss, int(gib * (1 << 27)))


def test_reused_then_returned(ara_lib):
    A = ara_lib
    ctx = A.ara_ctx_create(0)
    first = _table(A, ctx, 0.01)               # with it the runtime's own first allocations
    e = _table(A, ctx, 1.5)
    held = _free()
    A.ara_elt_release(e)
    assert abs(_free() - held) <= SLACK        # kept
    e = _table(A, ctx, 1.5)
    assert abs(_free() - held) <= SLACK        # and used again
    A.ara_elt_release(e)
    A.ara_set_option(ctx, A.ARA_OPT_KEPT_BYTES, GIB)
    assert _free() - held >= 1.4 * GIB         # more than the new limit: returned at once
    e = _table(A, ctx, 0.5)
    held = _free()
    A.ara_elt_release(e)
    assert abs(_free() - held) <= SLACK
    A.ara_set_option(ctx, A.ARA_OPT_KEPT_BYTES, 0)
    assert _free() - held >= 0.4 * GIB
    e = _table(A, ctx, 0.5)
    A.ara_elt_release(e)
    assert _free() - held >= 0.4 * GIB         # nothing kept any more
    for bad in (-1, (4 << 30) + 1):
        with pytest.raises(A.AraError):
            A.ara_set_option(ctx, A.ARA_OPT_KEPT_BYTES, bad)
    A.ara_elt_release(first)
    A.ara_ctx_destroy(ctx)


def test_returned_with_the_context(ara_lib):
    A = ara_lib
    for _ in range(2):                         # the first round loads the kernels
        before = _free()
        ctx = A.ara_ctx_create(0)
        A.ara_elt_release(_table(A, ctx, 1.5))
        kept = _free()
        A.ara_ctx_destroy(ctx)
    assert before - kept >= 1.4 * GIB
    assert before - _free() <= SLACK


def test_another_context_gets_what_one_keeps(ara_lib):
    import torch
    A = ara_lib
    one, other = A.ara_ctx_create(0), A.ara_ctx_create(0)
    A.ara_elt_release(_table(A, one, 1.9))
    hog = torch.empty(_free() - GIB, dtype=torch.uint8, device="cuda")     # 1 GiB left beside what `one` keeps
    try:
        e = _table(A, other, 1.9)
        A.ara_elt_release(e)
    finally:
        del hog
        torch.cuda.empty_cache()
        A.ara_ctx_destroy(other)
        A.ara_ctx_destroy(one)
