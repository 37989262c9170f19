"""Systems of one batch that end at different points of the iteration."""

import numpy as np
import pytest
import torch

from paper_2301_12836_amd import lsvie, models

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ell", [1, 2, 4])
@pytest.mark.parametrize("rel", [0.0, 1e-4, 0.2])
def test_batch_with_systems_that_end_early(ell, rel):
    """A zero right-hand side in the first slot, and systems that end at half steps (A = I without contrast: x = b after the
    first) and full steps.  Recurred and true residual differ by rounding only, at most 1e-6 of these tolerances; without
    contrast x carries two roundings.  Each system equals its own solve bit for bit."""
    m = models.random_medium((9, 6, 7), seed=4, rel=rel)
    ctx = lsvie.context_from_model(m, omegas=[2 * np.pi * 15.0], max_rhs=4, bicgstab_l=ell)
    b = torch.stack([ctx.rhs_moment(np.eye(6)[q], (2 + q, 2, 3)) for q in range(4)])
    b[0] = 0
    for tol in (0.3, 1e-2, 1e-5, 1e-9):
        # r_1 .. r_4 of an operator within 1e-4 of the identity differ by less than a rounding, so that the normal equations
        # of degree 4 are singular and whether their factorisation fails is chance: a reported breakdown is a right answer
        singular = (ell, rel, tol) == (4, 1e-4, 1e-9)
        u, infos = ctx.solve(b, tol=tol, maxit=300, raise_on_error=not singular)
        ok = torch.tensor([not (singular and i["status"] == lsvie.LS_ERR_BREAKDOWN) for i in infos], device=u.device)
        res = torch.linalg.vector_norm((b - ctx.apply(u)).reshape(4, -1), dim=1)
        nrm = torch.linalg.vector_norm(b.reshape(4, -1), dim=1)
        print(ell, rel, tol, [(i["iters"], i["matvecs"]) for i in infos], (res / nrm).tolist(), flush=True)
        assert torch.count_nonzero(u[0]) == 0 and infos[0]["iters"] == 0
        assert (res <= tol * (1 + 1e-6) * nrm)[ok].all()
        assert all(i["status"] == 0 for i, good in zip(infos, ok.tolist()) if good)
        if rel == 0.0:
            assert (torch.linalg.vector_norm((u - b).reshape(4, -1), dim=1) <= 4 * 2.0 ** -53 * nrm).all()
        for q in range(1, 4):
            single, info = ctx.solve(b[q], tol=tol, maxit=300, raise_on_error=not singular)
            assert torch.equal(single.reshape(u[q].shape), u[q]) and info[0]["status"] == infos[q]["status"], q
    ctx.close()
