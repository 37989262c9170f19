"""Tiles of the trace synthesis kernel."""

import numpy as np
import pytest
import torch

from paper_2301_12836_amd import lsvie, models

pytestmark = pytest.mark.gpu


# samples in tiles of 64, traces of 8, or of 16 from 256 tiles, frequencies in quarters; k n in 64 bits above 65536 samples;
# two launches above 2^20 samples or 16 x 65535 traces
@pytest.mark.parametrize("nf,ntr,nt", [(1, 1, 2), (2, 7, 63), (3, 8, 64), (4, 9, 65), (5, 1, 129), (33, 17, 800), (4, 315, 783), (3, 17, 8200), (9, 2, 65536),
                                       (9, 3, 65537), (2, 2, (1 << 20) + 3), (1, 16 * 65535 + 1, 2)])
def test_traces_match_the_sum_in_extended_precision(nf, ntr, nt):
    """Against the same sum with phases from exact integers.  A term carries at most ten roundings (phase, sine, wavelet
    factor, two products), the sum nf more: (nf + 10) unit roundoffs of the sum of magnitudes."""
    rng = np.random.default_rng(nf + ntr + nt)
    dt = 0.002
    k = np.sort(rng.choice(nt // 2 + 1, size=min(nf, nt // 2 + 1), replace=False))
    k[-1] = nt // 2
    U = rng.normal(size=(len(k), ntr)) + 1j * rng.normal(size=(len(k), ntr))
    ctx = lsvie.context_from_model(models.random_medium((4, 4, 4), seed=1), omegas=[60.0])
    got = ctx.synthesize(torch.from_numpy(U), k, nt, dt).cpu().numpy()
    ctx.close()
    c = np.where((k == 0) | (2 * k == nt), 1, 2) / (np.longdouble(nt) * np.longdouble(dt))
    ph = 2 * np.longdouble("3.14159265358979323846264338327950288") * ((k[:, None] * np.arange(nt)) % nt) / np.longdouble(nt)
    cu = c[:, None] * U.astype(np.clongdouble)
    want = cu.real.T @ np.cos(ph) + cu.imag.T @ np.sin(ph)
    bound = (len(k) + 10) * 2.0 ** -53 * np.abs(cu).sum(axis=0)[:, None]
    print(nf, ntr, nt, float((np.abs(got - want) / bound).max()), flush=True)
    assert got.shape == want.shape and (np.abs(got - want) <= bound).all()
