"""FFT lengths with factors 5, 7 and 9 along x and y (the z pass has its own file): both ends of the range of cells of
every length, solves whose inner products come from the x-inverse epilogue, the LDS Stockham kernels at those
lengths, and the limit of the allocation-free apply, which counts lengths 2^a and 3 2^a.

Tolerance of the applies: 100 unit roundoffs of the precision (relative L2): six transforms of at most nine radix-2
levels with two roundings each, and contrast sums of about thirty products."""

import numpy as np
import pytest
import torch

from oracle import operator as op
from paper_2301_12836_amd import lsvie, models

pytestmark = pytest.mark.gpu

EPS = {torch.complex128: 2.0 ** -53, torch.complex64: 2.0 ** -24}
W = 2 * np.pi * 12.0
N = [33, 40, 49, 56, 65, 72, 73, 80, 97, 112, 129, 144, 145, 160, 193, 224]   # 80, 112, 144, 160, 224, 288, 320, 448


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def check_apply(m, ctx):
    u = np.stack([models.random_field(m.shape, seed=s) for s in (1, 2)])
    P = op.Problem(m.shape, m.h, m.C0, m.rho0, m.dc21, m.drho, W)
    want = np.stack([P.apply_fft(x) for x in u])
    for dt in (torch.complex128, torch.complex64):
        e = rel(ctx.apply(torch.from_numpy(u).to(dt)).cpu().numpy(), want)
        print(m.shape, dt, e, flush=True)
        assert e < 100 * EPS[dt]


@pytest.mark.parametrize("n", N)
@pytest.mark.parametrize("axis", [0, 1])
def test_apply_at_every_xy_length(n, axis):
    shape = (n, 7, 5) if axis == 0 else (17, n, 5)
    m = models.random_medium(shape, seed=n, rel=0.1, aniso_background=True)
    ctx = lsvie.context_from_model(m, omegas=[W], precision="mixed", max_rhs=2)
    check_apply(m, ctx)
    ctx.close()


@pytest.mark.parametrize("n1", [40, 56, 72, 80, 112, 144, 160, 224])
def test_solve_with_fused_products(n1):
    m = models.random_medium((n1, 16, 8), seed=n1, rel=0.1, aniso_background=True)
    ctx = lsvie.context_from_model(m, omegas=[W], precision="mixed", max_rhs=2)
    b = np.stack([models.random_field(m.shape, seed=s) for s in (11, 12)])
    P = op.Problem(m.shape, m.h, m.C0, m.rho0, m.dc21, m.drho, W)
    for precision, tol in (("c128", 1e-10), ("mixed", 1e-6)):
        x, infos = ctx.solve(torch.from_numpy(b), tol=tol, maxit=2000, precision=precision)
        for r, v in enumerate(x.cpu().numpy()):
            res = rel(P.apply_fft(v), b[r])
            print(n1, precision, infos[r]["iters"], res, flush=True)
            assert infos[r]["status"] == 0 and res < 2 * tol
    ctx.close()


@pytest.mark.parametrize("shape", [(40, 56, 72), (80, 112, 33), (144, 9, 160), (8, 224, 193)])
def test_stockham_kernels(shape, tmp_path, monkeypatch):
    cache = tmp_path / "autotune.txt"
    monkeypatch.setenv("LS_AUTOTUNE_CACHE", str(cache))
    m = models.random_medium(shape, seed=sum(shape), rel=0.1, aniso_background=True)
    args = dict(omegas=[W], precision="mixed", max_rhs=2, autotune=True)
    lsvie.context_from_model(m, **args).close()
    key, *values = cache.read_text().split()
    cache.write_text(" ".join([key] + ["1"] * 10 + values[10:]) + "\n")
    ctx = lsvie.context_from_model(m, **args)
    assert all(v == "stockham" for p in ctx.kernel_variants.values() for v in p.values())
    check_apply(m, ctx)
    ctx.close()


@pytest.mark.parametrize("shape", [(40, 40, 40), (56, 56, 56), (65, 65, 65), (72, 8, 72)])
def test_noalloc_limit_counts_the_smooth_lengths(shape):
    L1, L2 = (min(v for v in (16, 32, 48, 64, 96, 128, 192, 256, 384, 512) if v >= 2 * n - 1) for n in shape[:2])
    fits = (64 << 20) // (3 * shape[2] * L2 * L1 * 16)   # the documented size per right-hand side
    m = models.random_medium(shape, seed=1, rel=0.1)
    ctx = lsvie.context_from_model(m, omegas=[W], max_rhs=8)
    u = torch.randn((8, 3) + shape[::-1], dtype=torch.complex128, device="cuda")
    out = torch.empty_like(u)
    for n in range(1, 9):
        if n <= fits:
            lsvie.ls_apply_noalloc(ctx.handle, 0, u, out, n)
            assert torch.equal(out[:n], ctx.apply(u[:n].contiguous()).reshape(out[:n].shape))
        else:
            with pytest.raises(lsvie.LsError):
                lsvie.ls_apply_noalloc(ctx.handle, 0, u, out, n)
    ctx.close()
