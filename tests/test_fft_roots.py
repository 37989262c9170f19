"""Every table of roots of unity in the FFT headers holds the doubles nearest to the cosines and sines it names."""

import os
import re
from fractions import Fraction

import pytest

from paper_2301_12836_amd import build

PI = Fraction("3.14159265358979323846264338327950288419716939937510582097494459230781640628620899862803482534")


def trig(m, n):
    """Nearest doubles of cos and sin of 2 pi m / n (0 <= m <= n / 2), from their power series in exact arithmetic."""
    x = 2 * PI * m / n
    c, s, term = Fraction(0), Fraction(0), Fraction(1)
    for k in range(60):   # x <= pi: the terms left out are below pi^60 / 60! < 1e-51
        if k % 2:
            s += term if k % 4 == 1 else -term
        else:
            c += term if k % 4 == 0 else -term
        term *= x / (k + 1)
    tiny = Fraction(1, 10 ** 40)
    return tuple(0.0 if abs(v) < tiny else float(v) for v in (c, s))


def tables():
    """(name, order, "c" or "s", values) of each table of cosines or sines."""
    for name in ("fft_core.h", "fft_reg.h"):
        with open(os.path.join(build.CSRC, name)) as f:
            text = re.sub(r"//[^\n]*", "", f.read())
        for struct, n, body in re.findall(r"struct (\w*Roots)<(\d+)> \{(.*?)\n\};", text, re.S):
            for kind, values in re.findall(r"double ([cs])\[\d+\] = \{(.*?)\}", body, re.S):
                yield f"{struct}<{n}>", int(n), kind, values
        for n, values in re.findall(r"double kCos(\d+)\[\d+\] = \{(.*?)\}", text, re.S):
            yield f"kCos{n}", int(n), "c", values


TABLES = list(tables())


def test_the_tables_are_found():
    assert {t[0] for t in TABLES} == {"OddRoots<5>", "OddRoots<7>", "Roots<9>", "Roots<10>", "Roots<14>", "kCos24", "kCos32"}


@pytest.mark.parametrize("name,n,kind,values", TABLES, ids=[f"{t[0]}.{t[2]}" for t in TABLES])
def test_roots_are_the_nearest_doubles(name, n, kind, values):
    got = [float(v) for v in values.split(",")]
    assert got == [trig(m, n)[kind == "s"] for m in range(len(got))]
