"""Incident fields of point sources in closed form, over the branches of the near-field term."""

import numpy as np
import pytest

from oracle import operator as op
from paper_2301_12836_amd import lsvie, models

pytestmark = pytest.mark.gpu


# h = 10 m, S speed 1730 m/s: w r / beta below 1/2 (the power series) at every cell; on both sides of it; above it at every
# cell but the source's own.
@pytest.mark.parametrize("w", [1.0, 40.0, 300.0])
@pytest.mark.parametrize("mode", ["exact", "paper_sum"])
@pytest.mark.parametrize("shape,src", [((2, 2, 2), (0, 0, 0)), ((17, 9, 5), (8, 4, 2)), ((33, 4, 19), (32, 3, 0))])
def test_incident_field_matches_the_oracle(shape, src, mode, w):
    """A general moment tensor and a force, inside and at a corner.  The terms lose up to about 20 of their size next to
    the border of the series (2 / (1/2)^2, and the difference of two such), the dipoles up to r / h = 20 more: 1000 unit
    roundoffs cover it."""
    m = models.random_medium(shape, seed=1)
    ctx = lsvie.context_from_model(m, omegas=[w], green_mode=mode)
    P = op.Problem(m.shape, m.h, m.C0, m.rho0, m.dc21, m.drho, w, mode=mode)
    M, F = [1.0, -0.4, 0.3, 0.7, -0.2, 0.5], [0.3, -1.0, 0.6]
    for got, want in ((ctx.rhs_moment(M, src, t0=0.004), P.rhs_moment(M, src, t0=0.004)),
                      (ctx.rhs_force(F, src), P.rhs_force(F, src))):
        e = float(np.linalg.norm(got.cpu().numpy() - want) / np.linalg.norm(want))
        print(shape, mode, w, e, flush=True)
        assert e < 1000 * 2.0 ** -53
    ctx.close()
