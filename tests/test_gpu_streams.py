"""Contexts on the null stream work on private streams: a dropped output's memory goes only to the same context."""

import pytest
import torch

from paper_2301_12836_amd import lsvie, models

pytestmark = pytest.mark.gpu


def test_dropped_outputs_are_reused_across_contexts():
    """The allocator hands the memory of a dropped output to the next call, which another context may make: every
    result is bitwise the one of the call alone."""
    shapes = [(40, 33, 24), (24, 40, 33)]
    ctxs, us, want = [], [], []
    for k, shape in enumerate(shapes):
        m = models.random_medium(shape, seed=k, rel=0.1)
        ctxs.append(lsvie.context_from_model(m, precision="mixed", max_rhs=3))
        us.append(torch.randn((3, 3) + shape[::-1], dtype=torch.complex64, device="cuda"))
        want.append(ctxs[k].apply(us[k]))
    torch.cuda.synchronize()
    for _ in range(50):
        ctxs[0].apply(us[0])
        ctxs[1].apply(us[1])
        a = ctxs[0].apply(us[0])
        ctxs[1].apply(us[1])
        torch.cuda.synchronize()
        assert torch.equal(a, want[0])
        a = ctxs[1].apply(us[1])
        ctxs[0].apply(us[0])
        b = ctxs[1].apply(us[1])
        torch.cuda.synchronize()
        assert torch.equal(a, want[1]) and torch.equal(b, want[1])
    for c in ctxs:
        c.close()


def test_outputs_come_from_the_context_stream():
    m = models.random_medium((8, 9, 10), seed=1, rel=0.1)
    a, b = lsvie.context_from_model(m), lsvie.context_from_model(m)
    u = torch.randn(a.field_shape, dtype=torch.complex128, device="cuda")
    ptr = a.apply(u).data_ptr()        # dropped at once
    assert b.apply(u).data_ptr() != ptr and a.apply(u).data_ptr() == ptr
    assert torch.cuda.current_stream().cuda_stream == 0
    a.close()
    b.close()


def test_solve_after_an_asynchronous_call():
    """b = A v written by an apply is the right-hand side of the next solve, through the same workspace."""
    m = models.random_medium((48, 40, 36), seed=3, rel=0.05)
    ctx = lsvie.context_from_model(m, max_rhs=2)
    v = torch.randn((2,) + ctx.field_shape, dtype=torch.complex128, device="cuda")
    for _ in range(3):
        x, infos = ctx.solve(ctx.apply(v), tol=1e-12)
        y = ctx.apply(x)
        assert all(i["status"] == 0 for i in infos)
        assert (torch.linalg.vector_norm(x - v) / torch.linalg.vector_norm(v)).item() < 1e-10
        assert (torch.linalg.vector_norm(y - ctx.apply(v)) / torch.linalg.vector_norm(y)).item() < 1e-11
    ctx.close()
