"""The strain and gradient kernels on grids that end one cell short of a block of 256 cells, at its end and one cell into
the next, over block counts that do and do not divide among the XCDs."""

import numpy as np
import pytest
import torch

from oracle import operator as op
from paper_2301_12836_amd import lsvie, models

pytestmark = pytest.mark.gpu

# 20, 255, 256, 513, 1023, 1281 and 2048 cells; 40 blocks and one cell
SHAPES = [(5, 2, 2), (3, 5, 17), (16, 8, 2), (3, 3, 57), (3, 11, 31), (3, 7, 61), (16, 16, 8), (49, 11, 19)]
W = 60.0


def fields(shape, seeds):
    return np.stack([models.random_field(shape, seed=s) for s in seeds])


def context(m, r):
    return lsvie.context_from_model(m, omegas=[W], max_rhs=r)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("r", [1, 3])
def test_strain(shape, r):
    """Three-point differences and sums of two: at most ten roundings of the largest strain."""
    m = models.random_medium(shape, seed=1)
    ctx = context(m, r)
    u = fields(shape, range(r))
    got = ctx.strain(torch.from_numpy(u).to(ctx.device)).cpu().numpy().reshape(r, 6, *shape[::-1])
    ctx.close()
    for q in range(r):
        want = op.strain_apply(u[q], m.h)
        assert float(np.abs(got[q] - want).max() / np.abs(want).max()) < 10 * 2.0 ** -53


def gradient(u, mu, h):
    """dJ/d(dC) and dJ/d(drho) of fields u and mu, and the largest sums of absolute terms."""
    n = u.shape[-3:]
    g, gr, top = np.zeros((21,) + n), np.zeros(n), [0.0, 0.0]
    for a, b in zip(u, mu):
        ea, eb = op.strain_apply(a, h), op.strain_apply(b, h)
        q = 0
        for i in range(6):
            for j in range(i, 6):
                v = np.conj(eb[i]) * ea[j]
                g[q] -= (v + np.conj(eb[j]) * ea[i] if i != j else v).real
                q += 1
        gr += W * W * (np.conj(b) * a).real.sum(0)
        top[0] += 4 * np.abs(ea).max() * np.abs(eb).max()
        top[1] += 6 * W * W * np.abs(a).max() * np.abs(b).max()
    return g, gr, top


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("r", [1, 3])
def test_gradients(shape, r):
    """From mu as given, and through the conjugated form with mu the conjugate of the convolved field.  Strains carry ten
    roundings each, a sum of at most four products per field as many again: within 40 of the largest sum of terms."""
    m = models.random_medium(shape, seed=1)
    ctx = context(m, r)
    u, lam = fields(shape, range(r)), fields(shape, range(10, 10 + r))
    mu = ctx.convolve(torch.from_numpy(lam)).conj().resolve_conj()
    want = gradient(u, mu.cpu().numpy().reshape(u.shape), m.h)
    for got in (ctx.grad_contrast(torch.from_numpy(u), mu), ctx.grad(torch.from_numpy(u), torch.from_numpy(lam))[:2]):
        for x, w, top in zip(got, want[:2], want[2]):
            e = float(np.abs(x.cpu().numpy() - w).max() / top)
            print(shape, r, e, flush=True)
            assert e < 40 * 2.0 ** -53
    ctx.close()
