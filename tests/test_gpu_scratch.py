"""Device memory of a context: the tables that the first plan with symmetric
tiles adds take four words per particle, in either precision (the low words of
the FP64 totals lie in rows that the context holds in any case)."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("prec", [0, 1])
def test_symmetric_tables(prec):
    import paper_2506_06269_amd as S
    n = 1 << 20
    dev = S.state_to_device(W.nfw_halo(n, seed=1))
    # the same kernels on another context first: what the runtime itself takes
    # for their code and their private memory is not the context's
    ctx = S.sidm_create(0, 1 << 17, 1)
    S.sidm_gravity(ctx, [dict(n=1 << 17, eps=0.01)], dev, prec)
    S.sidm_destroy(ctx)
    ctx = S.sidm_create(0, n, 1)
    before = _free()
    S.sidm_gravity(ctx, [dict(n=n, eps=0.01)], dev, prec)
    grown = before - _free()
    S.sidm_destroy(ctx)
    print(f"{grown / n:.1f} B per particle", flush=True)
    # the totals, and 8 B for the work items and the granularity of allocations
    assert grown <= (32 + 8) * n


def test_more_events_keep_the_candidates():
    """Raising the event capacity does not lower the number of candidates (two
    per particle of 80 bytes in a new context)."""
    import paper_2506_06269_amd as S
    n = 1 << 22
    _free()   # torch's runtime first
    ctx = S.sidm_create(0, n, 1)
    before = _free()
    S.sidm_set_event_capacity(ctx, n // 4)
    assert _free() <= before
    S.sidm_destroy(ctx)
