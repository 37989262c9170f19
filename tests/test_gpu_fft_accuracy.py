"""FP32 applications at FFT lengths with a factor 7 or 9 round no more than at the next power of two.

The DFTs of length 7, 9 and 14 sum in FP64 and round once or twice, the radix-8 and radix-16 DFTs in their place at a power of
two three or four times, and both lines take one more DFT and one product with twiddles.  So the relative L2 error of an
application, against FP64 on the same inputs, is at most the one at the power of two with the same share of padding."""

import pytest
import torch

from paper_2301_12836_amd import lsvie, models

pytestmark = pytest.mark.gpu


def error(n):
    m = models.random_medium((n, n, n), seed=n, rel=0.1)
    ctx = lsvie.context_from_model(m, omegas=[60.0], precision="mixed", max_rhs=2)
    gen = torch.Generator(device="cuda").manual_seed(n)
    u = torch.randn((2, 3, n, n, n), dtype=torch.complex64, device="cuda", generator=gen)
    want = ctx.apply(u.to(torch.complex128))
    e = torch.linalg.vector_norm(ctx.apply(u).to(torch.complex128) - want) / torch.linalg.vector_norm(want)
    ctx.close()
    return e.item()


@pytest.mark.parametrize("n,power", [(56, 64), (72, 64), (112, 128), (144, 128)])   # lengths 112, 144, 224, 288
def test_odd_factors_round_no_more_than_powers_of_two(n, power):
    e, ref = error(n), error(power)
    print(n, e, power, ref, flush=True)
    assert e <= ref
