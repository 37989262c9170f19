"""BiCGSTAB(l) on operators so close to the identity that the residuals of a cycle are linearly dependent to rounding:
every solve reaches its tolerance."""

import numpy as np
import pytest
import torch

from paper_2301_12836_amd import lsvie, models

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ell", [2, 3, 4])
@pytest.mark.parametrize("rel", [0.0, 1e-7, 1e-5, 1e-4, 1e-3, 1e-2])
@pytest.mark.parametrize("precision", ["c128", "mixed"])
def test_solves_near_the_identity(ell, rel, precision):
    """Recurred and true residual differ by rounding only: at most 1e-6 of these tolerances in FP64."""
    m = models.random_medium((9, 6, 7), seed=4, rel=rel)
    ctx = lsvie.context_from_model(m, omegas=[2 * np.pi * 15.0], precision="mixed", max_rhs=4, bicgstab_l=ell)
    b = torch.stack([ctx.rhs_moment(np.eye(6)[q], (2 + q, 2, 3)) for q in range(4)])
    nrm = torch.linalg.vector_norm(b.reshape(4, -1), dim=1)
    for tol in (1e-5, 1e-7, 1e-9, 1e-12):
        for solve, op in ((ctx.solve, ctx.apply), (ctx.solve_T, ctx.apply_T)):
            u, infos = solve(b, tol=tol, maxit=300, precision=precision)
            res = torch.linalg.vector_norm((b - op(u)).reshape(4, -1), dim=1) / nrm
            print(ell, rel, precision, tol, [(i["iters"], i["matvecs"]) for i in infos], res.tolist(), flush=True)
            assert all(i["status"] == 0 for i in infos)
            assert (res <= tol * (1 + 1e-6) + 2.0 ** -50).all()
    ctx.close()


@pytest.mark.parametrize("ell", [2, 4])
@pytest.mark.parametrize("rel", [1e-5, 1e-3])
def test_a_tolerance_below_rounding_ends(ell, rel):
    """The solve ends (the recurred residual may fall below rounding, and the status goes by it) and leaves a field whose true
    residual is rounding: within 2^13 unit roundoffs."""
    m = models.random_medium((9, 6, 7), seed=4, rel=rel)
    ctx = lsvie.context_from_model(m, omegas=[2 * np.pi * 15.0], max_rhs=2, bicgstab_l=ell)
    b = torch.stack([ctx.rhs_moment(np.eye(6)[q], (2 + q, 2, 3)) for q in range(2)])
    u, infos = ctx.solve(b, tol=1e-19, maxit=200, raise_on_error=False)
    res = torch.linalg.vector_norm((b - ctx.apply(u)).reshape(2, -1), dim=1) / torch.linalg.vector_norm(b.reshape(2, -1), dim=1)
    print(ell, rel, [(i["status"], i["iters"]) for i in infos], res.tolist(), flush=True)
    assert all(i["iters"] <= 200 for i in infos)
    assert (res < 2.0 ** -40).all()
    ctx.close()
