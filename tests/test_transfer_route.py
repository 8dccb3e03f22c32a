"""Which kernel a coarse-to-fine transfer takes, and that the marching kernel's
taps and launch are those of the stencils wherever it applies (host rules on
the CPU under AddressSanitizer and UBSan)."""
import os
import subprocess
import tempfile

import pytest

from tests.harness_util import ROOT

_EXE = []


def routes(cases):
    """Per (coarse (z, y, x), fine (z, y, x), element size, tallest band): for u,
    v, w (rows, taken, taps right, general kernel piped)."""
    if not _EXE:
        exe = os.path.join(tempfile.mkdtemp(prefix="ch_route_"), "route_dump")
        subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=undefined", "-fno-omit-frame-pointer", "-o", exe,
                        os.path.join(ROOT, "tests", "cpu_harness", "route_dump.cpp")], check=True)
        _EXE.append(exe)
    text = "".join(" ".join(map(str, (*nc, *nf, es, rmax))) + "\n" for nc, nf, es, rmax in cases)
    r = subprocess.run([_EXE[0]], input=text, capture_output=True, text=True,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, r.stderr
    out = []
    for line in r.stdout.splitlines():
        v = list(map(int, line.split()))
        out.append([tuple(v[4 * c:4 * c + 4]) for c in range(3)])
    assert len(out) == len(cases)
    return out


@pytest.mark.parametrize("nc,nf,es,rmax,rows,taken", [
    # two fine cells per coarse one: always
    ((8, 8, 8), (16, 16, 16), 4, 20, 8, True),
    ((8, 8, 8), (16, 16, 16), 8, 20, 8, True),
    ((256, 256, 256), (512, 512, 512), 8, 20, 8, True),
    # selected taps: from 192 groups on
    ((24, 64, 64), (32, 192, 192), 4, 15, 8, False),
    ((64, 64, 64), (192, 192, 192), 4, 15, 8, True),
    ((64, 64, 64), (192, 192, 192), 8, 15, 8, True),
    # eleven rows in double precision: up to 128 points, or odd target rows
    ((128, 128, 128), (192, 192, 192), 8, 25, 11, True),
    ((160, 256, 256), (240, 384, 384), 8, 15, 11, False),
    # ... and where the last round of 256 groups is at least two thirds of the CUs
    ((64, 96, 96), (96, 152, 152), 8, 24, 11, True),       # 240 groups
    ((64, 96, 96), (128, 152, 152), 8, 24, 11, False),     # 320
    ((64, 128, 128), (128, 192, 192), 8, 25, 11, True),    # 384
    ((24, 128, 256), (44, 192, 385), 8, 15, 11, False),    # 264, odd target rows
    ((160, 256, 256), (272, 435, 435), 8, 15, 11, True),
    # eleven rows in single precision: large piped shapes stay
    ((96, 256, 256), (144, 384, 384), 4, 16, 11, True),
    ((160, 256, 256), (240, 384, 384), 4, 16, 11, False),
    ((200, 200, 200), (340, 340, 340), 4, 24, 11, True),
    # coarse rows or target rows the kernel does not hold
    ((64, 300, 300), (128, 600, 600), 4, 20, 0, False),
    ((60, 256, 256), (120, 1040, 1100), 4, 12, 0, False),
    ((64, 256, 256), (64, 256, 256), 4, 20, 0, False),
])
def test_route(nc, nf, es, rmax, rows, taken):
    (r,) = routes([(nc, nf, es, rmax)])
    assert max(c[0] for c in r) == rows
    assert all(c[1] == taken for c in r)


def test_marching_taps_are_the_stencils_wherever_it_applies():
    cases = [((8, cy, cx), (16, fy, fx), es, 12)
             for cx in (4, 5, 6, 7, 8, 12, 37, 63, 64, 65, 128, 129, 256)
             for fx in (8, 9, 10, 16, 18, 63, 64, 100, 128, 256, 257, 400, 512, 1024)
             for cy, fy in ((4, 8), (5, 13), (cx, fx)) for es in (4, 8)]
    got = routes(cases)
    for case, r in zip(cases, got):
        assert all(c[2] == 1 for c in r), case
        # the general kernel keeps its loads a whole item ahead where it did
        assert all(c[3] == (case[3] <= (20 if case[2] == 4 else 12) and case[0][2] <= 256)
                   for c in r)
    assert 100 < sum(c[0] > 0 for r in got for c in r)
