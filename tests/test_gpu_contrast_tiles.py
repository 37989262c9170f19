"""The tiles and z chunks of the fused contrast kernel."""

import numpy as np
import pytest
import torch

from oracle import operator as op
from paper_2301_12836_amd import lsvie, models

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(2, 2, 2), (16, 8, 3), (17, 9, 2), (31, 4, 5), (33, 15, 7), (48, 8, 9), (101, 100, 100),
                                   (97, 104, 102), (136, 90, 90)])
def test_tiles_and_chunks_of_the_fused_contrast(shape):
    """Both FP32 tiles (narrow up to a million cells or where it covers a fifth fewer), the FP64 tile and z chunks down to
    single planes: the operator equals the oracle's within 100 unit roundoffs (see test_gpu_lengths)."""
    m = models.random_medium(shape, seed=sum(shape), rel=0.1, aniso_background=True)
    w = 2 * np.pi * 12.0
    ctx = lsvie.context_from_model(m, omegas=[w], precision="mixed", max_rhs=1)
    u = models.random_field(m.shape, seed=3)
    want = op.Problem(m.shape, m.h, m.C0, m.rho0, m.dc21, m.drho, w).apply_fft(u)
    for dt, eps in ((torch.complex128, 2.0 ** -53), (torch.complex64, 2.0 ** -24)):
        got = ctx.apply(torch.from_numpy(u).to(dt)).cpu().numpy()
        e = float(np.linalg.norm(got - want) / np.linalg.norm(want))
        print(shape, dt, e, flush=True)
        assert e < 100 * eps
    ctx.close()
