"""Contexts on the default stream pass fields on to one another, and memory that the allocator hands out again, without
waiting: each call sees what the calls before it wrote and changes nothing that they still read.

Every result is bitwise the one of the same calls with a device synchronisation after each."""

import threading

import numpy as np
import pytest
import torch

from paper_2301_12836_amd import lsvie, models

pytestmark = pytest.mark.gpu

SHAPE = (72, 64, 56)   # an application takes several times a call's host time


def contexts(n, shape=SHAPE, rel=0.05, **kw):
    return [lsvie.context_from_model(models.random_medium(shape, seed=k, rel=rel), omegas=[60.0], max_rhs=2, **kw) for k in range(n)]


def field(seed, shape=SHAPE, n=2, dtype=torch.complex128):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn((n, 3) + shape[::-1], dtype=dtype, device="cuda", generator=gen)


def synced(f, *args, **kw):
    torch.cuda.synchronize()
    out = f(*args, **kw)
    torch.cuda.synchronize()
    return out


def check(got, want):
    torch.cuda.synchronize()
    assert torch.equal(got, want)


CALLS = {
    "apply": lambda c, u: c.apply(u),
    "apply_T": lambda c, u: c.apply_T(u),
    "convolve": lambda c, u: c.convolve(u),
    "strain": lambda c, u: c.strain(u),
    "grad_contrast": lambda c, u: c.grad_contrast(u, u)[0],
    "grad": lambda c, u: c.grad(u, u)[0],
    "solve": lambda c, u: c.solve(u, tol=1e-3, maxit=400)[0],
    "sample": lambda c, u: c.sample(u, np.array([[0, 0, 0], [5, 6, 7], [71, 63, 55]])),
}


@pytest.mark.parametrize("name", CALLS)
def test_a_field_passed_on(name):
    a, b = contexts(2)
    us = [field(k) for k in range(4)]
    want = [synced(CALLS[name], b, synced(a.apply, u)) for u in us]
    for _ in range(3):
        for u, w in zip(us, want):
            check(CALLS[name](b, a.apply(u)), w)
    a.close()
    b.close()


def test_a_field_passed_on_in_fp32():
    a, b = contexts(2, precision="mixed")
    u = field(1, dtype=torch.complex64)
    want = synced(b.apply, synced(a.apply, u))
    for _ in range(5):
        check(b.apply(a.apply(u)), want)
    a.close()
    b.close()


def test_a_passed_on_field_dropped_while_it_is_read():
    """y of A goes to B and is dropped: the next output of A takes its memory."""
    a, b = contexts(2)
    us = [field(k) for k in range(6)]
    want = [synced(b.apply, synced(a.apply, u)) for u in us]
    zs = []
    for u in us:
        y = a.apply(u)
        zs.append(b.apply(y))
        del y
    torch.cuda.synchronize()
    for z, w in zip(zs, want):
        assert torch.equal(z, w)
    a.close()
    b.close()


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
def test_an_input_dropped_while_it_is_read(dtype):
    """A's input, or the converted copy of one, is dropped: B's incident field takes its memory."""
    a, b = contexts(2)
    us = [field(k, n=1, dtype=dtype)[0] for k in range(4)]
    want = [synced(a.apply_T, u) for u in us]
    for _ in range(3):
        for u, w in zip(us, want):
            y = a.apply_T(u.clone())
            rhs = [b.rhs_moment([1, 2, 3, 0, 0, 0], (9, 9, 9)) for _ in range(2)]
            check(y, w)
            del rhs
    a.close()
    b.close()


def test_accumulators_shared_by_two_contexts():
    a, b = contexts(2)
    u, v = field(1), field(2)
    g, r = synced(a.grad_contrast, u, v)
    g, r = synced(b.grad, u, v, g_dC=g, g_drho=r)[:2]
    for _ in range(3):
        p, q = a.grad_contrast(u, v)
        p, q = b.grad(u, v, g_dC=p, g_drho=q)[:2]
        check(p, g)
        check(q, r)
    a.close()
    b.close()


def test_the_allocation_free_apply_on_two_contexts():
    """Its work buffer is one array for both."""
    shape = (40, 36, 33)
    a, b = contexts(2, shape)
    u = field(1, shape)
    want = [synced(c.apply, u) for c in (a, b)]
    outs = [torch.empty_like(u) for _ in range(2)]
    torch.cuda.synchronize()
    for _ in range(10):
        for c, out in zip((a, b), outs):
            lsvie.ls_apply_noalloc(c.handle, 0, u, out, 2)
    for out, w in zip(outs, want):
        check(out, w)
    a.close()
    b.close()


def test_more_calls_in_flight_than_ranges_are_kept():
    """A chain over three contexts through 150 buffers of one block of memory, near the identity."""
    shape = (12, 10, 9)
    ctxs = contexts(3, shape, rel=0.01)
    pool = torch.empty((150, 3) + shape[::-1], dtype=torch.complex128, device="cuda")

    def apply(k, i, o):
        lsvie.ls_apply(ctxs[k % 3].handle, 0, pool[i], pool[o], 1)

    def chain(after):
        pool.zero_()
        pool[0] = field(3, shape, 1)[0]
        for k in range(149):
            apply(k * 7, k, k + 1)
            after()
            if k % 4 == 3:   # memory that another context has read and written
                apply(k, k + 1, k - 3)
                after()
        torch.cuda.synchronize()
        return pool.clone()

    want = chain(torch.cuda.synchronize)
    assert torch.isfinite(torch.view_as_real(want)).all()
    for _ in range(5):
        assert torch.equal(chain(lambda: None), want)
    for c in ctxs:
        c.close()


def test_a_field_read_in_another_thread_while_its_context_records_a_graph():
    a, b = contexts(2)
    u, rhs = field(1), field(2)
    w, y, x = (torch.empty_like(u) for _ in range(3))
    want_y = synced(b.apply_T, synced(a.apply, u))
    want_x = synced(a.solve, rhs, tol=1e-6)[0]
    for _ in range(4):
        for t in (w, x, y):
            t.zero_()
        a.apply(u, out=w)
        solve = threading.Thread(target=lambda: a.solve(rhs, tol=1e-6, out=x))
        solve.start()
        for _ in range(20):
            lsvie.ls_apply_T(b.handle, 0, w, y, 2)
        solve.join()
        check(x, want_x)
        check(y, want_y)
    a.close()
    b.close()


def test_a_batch_after_calls_that_still_run():
    a, b = contexts(2)
    jobs = [(k % 2, 0, [1, 1, 1, 0, 0, k], (20 + k, 30, 28), 0.0) for k in range(4)]
    want, _ = synced(lsvie.solve_batch, [a, b], jobs, tol=1e-4)
    us = [field(k, n=1)[0] for k in range(4)]
    w = [synced(b.convolve, synced(a.apply, u)) for u in us]
    for _ in range(3):
        outs = [torch.empty_like(u) for u in us]
        zs = [b.convolve(a.apply(u, out=o)) for u, o in zip(us, outs)]   # b reads outs while the batch writes them
        got, _ = lsvie.solve_batch([a, b], jobs, tol=1e-4, outs=outs)
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(got, want))
        assert all(torch.equal(x, y) for x, y in zip(zs, w))
    a.close()
    b.close()
