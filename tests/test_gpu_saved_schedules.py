"""Saved kernel choices that were timed with the kernels of another build are not taken."""

import re

import numpy as np
import pytest

from paper_2301_12836_amd import lsvie, models

pytestmark = pytest.mark.gpu

STOCKHAM = " 1 1 1 1 1 1 1 1 1 1 1 1 0 0\n"


def tuned(m):
    return lsvie.context_from_model(m, omegas=[2 * np.pi * 12.0], precision="mixed", max_rhs=2, autotune=True)


@pytest.mark.parametrize("older", [r"v2:", r"v2:k1:"])
def test_choices_timed_with_other_kernels_are_not_taken(older, tmp_path, monkeypatch):
    cache = tmp_path / "autotune.txt"
    monkeypatch.setenv("LS_AUTOTUNE_CACHE", str(cache))
    m = models.random_medium((24, 20, 18), seed=1, rel=0.1)
    tuned(m).close()
    key = cache.read_text().split()[0]
    saved = re.sub(r"^v2:(k\d+:)?", older, key) + STOCKHAM
    cache.write_text(saved)
    tuned(m).close()
    assert cache.read_text().startswith(saved) and cache.read_text().count("\n") == 2   # tuned, and saved beside it
