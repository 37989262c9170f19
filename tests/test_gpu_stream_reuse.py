"""Private streams go from closed contexts to new ones, with the memory that the allocator keeps for them."""

import pytest
import torch

from paper_2301_12836_amd import lsvie, models

pytestmark = pytest.mark.gpu

SHAPE = (40, 36, 32)


def context(seed=1, shape=SHAPE, **kw):
    return lsvie.context_from_model(models.random_medium(shape, seed=seed, rel=0.1), omegas=[60.0], **kw)


def test_new_contexts_take_the_streams_of_closed_ones():
    first = [context(k, (6, 5, 4)) for k in range(5)]
    streams = {lsvie.ls_stream(c.handle) for c in first}
    assert len(streams) == 5
    for c in first:
        c.close()
    for _ in range(3):
        again = [context(k, (6, 5, 4)) for k in range(5)]
        assert {lsvie.ls_stream(c.handle) for c in again} == streams
        for c in again:
            c.close()


def test_contexts_in_a_loop_find_the_memory_of_dropped_outputs():
    """The next context is open before the last one closes; each makes fields and gradients."""
    u = torch.randn((3,) + SHAPE[::-1], dtype=torch.complex128, device="cuda")
    reserved, old = [], context()
    for k in range(10):
        new = context(k)
        outs = [old.apply(u), old.strain(u), *old.grad(u, u)[:2]]
        torch.cuda.synchronize()
        del outs
        old.close()
        old = new
        reserved.append(torch.cuda.memory_reserved())
    old.close()
    assert max(reserved[2:]) <= reserved[2]


def test_outputs_outlive_their_context():
    ctx = context()
    u = torch.randn((3,) + SHAPE[::-1], dtype=torch.complex128, device="cuda")
    y = ctx.apply(u)
    torch.cuda.synchronize()
    want = y.clone()
    ctx.close()
    other = context()
    for _ in range(4):
        other.apply(u + 1)
    torch.cuda.synchronize()
    assert torch.equal(y, want)
    del y
    other.close()


def test_calls_of_a_closed_context_are_refused():
    """Also those whose outputs are cleared before the library sees the call."""
    ctx = context()
    u = torch.randn((3,) + SHAPE[::-1], dtype=torch.complex128, device="cuda")
    ctx.apply(u)
    ctx.close()
    for call in (ctx.apply, ctx.strain, ctx.convolve, lambda v: ctx.grad(v, v), lambda v: ctx.grad_contrast(v, v)):
        with pytest.raises(lsvie.LsError):
            call(u)
    torch.cuda.synchronize()


@pytest.mark.parametrize("failures", [1, 2])
def test_a_setup_without_memory_is_tried_again_without_the_cache(failures, monkeypatch):
    torch.empty(1 << 26, dtype=torch.uint8, device="cuda")   # dropped: stays in the cache
    setup, reserved = lsvie.ls_setup, []

    def limited(*args, **kw):
        reserved.append(torch.cuda.memory_reserved())
        if len(reserved) <= failures:
            raise lsvie.LsError(lsvie.LS_ERR_OOM, "no memory left")
        return setup(*args, **kw)

    monkeypatch.setattr(lsvie, "ls_setup", limited)
    if failures == 2:
        with pytest.raises(lsvie.LsError):
            context()
    else:
        context().close()
    assert len(reserved) == 2 and reserved[1] <= reserved[0] - (1 << 26)
