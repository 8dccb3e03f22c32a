"""The transforms' twiddles against values of 50 decimal digits: within 0.51 units
in the last place (once rounded; the extended-precision sine behind them may add
a little)."""
import os
import subprocess
import tempfile
from decimal import Decimal, getcontext

import numpy as np
import pytest

from tests.harness_util import ROOT

_EXE = []
PI = Decimal("3.14159265358979323846264338327950288419716939937510582097494459")


def _sincos(x):
    """sin and cos of a Decimal by their series."""
    getcontext().prec = 50
    s = c = Decimal(0)
    t, k = Decimal(1), 0
    while abs(t) > Decimal(10) ** -45 or k < 4:
        c, s = (c + t * (1 if k % 4 == 0 else -1), s) if k % 2 == 0 else \
            (c, s + t * (1 if k % 4 == 1 else -1))
        k += 1
        t = t * x / k
    return s, c


@pytest.mark.parametrize("n", [2, 3, 8, 27, 100, 240, 512, 625, 1000, 1024])
def test_twiddles_are_rounded_once(n):
    if not _EXE:
        exe = os.path.join(tempfile.mkdtemp(prefix="ch_twiddle_"), "twiddle_dump")
        subprocess.run(["g++", "-O2", "-std=c++17", "-o", exe,
                        os.path.join(ROOT, "tests", "cpu_harness", "twiddle_dump.cpp")], check=True)
        _EXE.append(exe)
    r = subprocess.run([_EXE[0]], input=f"{n}\n", capture_output=True, text=True, check=True)
    got = np.array(r.stdout.split(), dtype=np.float64).reshape(n, 2)
    for m in range(n):
        s, c = _sincos(2 * PI * m / n)
        for g, want in ((got[m, 0], c), (got[m, 1], -s)):
            # zeros of the sine and cosine: the angle's own rounding, 2^-64 of 2 pi
            ulp = Decimal(float(np.spacing(abs(float(want))))) if abs(want) > Decimal("1e-15") \
                else Decimal("1e-17")
            assert abs(Decimal(float(g)) - want) <= Decimal("0.51") * ulp + Decimal("7e-19"), (n, m)
