"""The strain kernel over grids whose blocks do not divide among the XCDs."""

import numpy as np
import pytest
import torch

from oracle import operator as op
from paper_2301_12836_amd import lsvie, models

pytestmark = pytest.mark.gpu


# 8 cells; one block exactly, one cell more; 8 blocks and one cell more; ragged
@pytest.mark.parametrize("shape", [(2, 2, 2), (16, 8, 2), (257, 1, 1), (16, 16, 8), (2, 5, 205), (50, 41, 37)])
@pytest.mark.parametrize("r", [1, 3])
def test_strain_matches_the_oracle(shape, r):
    """Three-point differences and sums of two: at most ten roundings of the largest strain."""
    shape = tuple(min(max(n, 2), 256) for n in shape)
    m = models.random_medium(shape, seed=1)
    ctx = lsvie.context_from_model(m, omegas=[60.0], max_rhs=r)
    u = np.stack([models.random_field(m.shape, seed=q) for q in range(r)])
    got = ctx.strain(torch.from_numpy(u).to(ctx.device)).cpu().numpy().reshape(r, 6, *shape[::-1])
    ctx.close()
    for q in range(r):
        want = op.strain_apply(u[q], m.h)
        e = float(np.abs(got[q] - want).max() / np.abs(want).max())
        print(shape, r, e, flush=True)
        assert e < 10 * 2.0 ** -53
