"""The LDS z kernel with a half-space table, as a saved choice selects it and tables above 4 GB take it."""

import numpy as np
import pytest
import torch

from paper_2301_12836_amd import lsvie, models

pytestmark = pytest.mark.gpu

EPS = {torch.complex128: 2.0 ** -53, torch.complex64: 2.0 ** -24}
STOCKHAM = " 1 1 1 1 1 1 1 1 1 1 1 1 0 0\n"


def tuned(m, **kw):
    return lsvie.context_from_model(m, omegas=[2 * np.pi * 12.0], precision="mixed", max_rhs=2, autotune=True, **kw)


@pytest.mark.parametrize("n3", [2, 8, 13, 24, 40, 56, 72, 96, 112, 129, 160, 256])
def test_lds_z_kernel_with_a_half_space_table(n3, tmp_path, monkeypatch):
    """A mirror-symmetric background through the half-space table gives the operator of the octant table: within 100 unit
    roundoffs (relative L2; six transforms of at most nine radix-2 levels with two roundings each, and contrast sums of
    about thirty products)."""
    cache = tmp_path / "autotune.txt"
    monkeypatch.setenv("LS_AUTOTUNE_CACHE", str(cache))
    m = models.random_medium((5, 4, n3), seed=n3, rel=0.1, aniso_background=True)
    octant = lsvie.context_from_model(m, omegas=[2 * np.pi * 12.0], precision="mixed", max_rhs=2, green_mode="aniso")
    monkeypatch.setenv("LS_GREEN_TABLE", "half")
    tuned(m, green_mode="aniso").close()
    cache.write_text(cache.read_text().split()[0] + STOCKHAM)
    half = tuned(m, green_mode="aniso")
    assert all(v == "stockham" for p in half.kernel_variants.values() for v in p.values())
    u = torch.from_numpy(np.stack([models.random_field(m.shape, seed=s) for s in (1, 2)]))
    for dt in (torch.complex128, torch.complex64):
        a, b = half.apply(u.to(dt)), octant.apply(u.to(dt))
        e = (torch.linalg.vector_norm(a - b) / torch.linalg.vector_norm(b)).item()
        print(n3, dt, e, flush=True)
        assert e < 100 * EPS[dt]
    octant.close()
    half.close()
