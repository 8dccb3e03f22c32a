"""Which transforms a pressure solve takes (its own or the FFT library's), their
radices and the spectrum's row pitch: the host rules on the CPU under
AddressSanitizer and UBSan."""
import os
import subprocess
import tempfile

import numpy as np
import pytest

from tests.harness_util import ROOT

_EXE = []


def route(cases):
    """Per (shape (z, y, x), walls, FP32): own, pitch, radices per axis x, y, z."""
    if not _EXE:
        exe = os.path.join(tempfile.mkdtemp(prefix="ch_poisson_"), "poisson_dump")
        subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=undefined", "-fno-omit-frame-pointer", "-o", exe,
                        os.path.join(ROOT, "tests", "cpu_harness", "poisson_dump.cpp")], check=True)
        _EXE.append(exe)
    text = "".join(f"{s[2]} {s[1]} {s[0]} {int(w)} {int(p)}\n" for s, w, p in cases)
    r = subprocess.run([_EXE[0]], input=text, capture_output=True, text=True,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, r.stderr
    out = []
    for line in r.stdout.splitlines():
        v = list(map(int, line.split()))
        radices, k = [], 2
        for _ in range(3):
            radices.append(v[k + 1:k + 1 + v[k]])
            k += 1 + v[k]
        out.append((bool(v[0]), v[1], radices))
    return out


@pytest.mark.parametrize("shape,walls,pitch", [
    # own transforms: whole cache lines from 16 elements on
    ((160, 180, 240), 0, 128), ((27, 27, 27), 0, 14), ((36, 64, 36), 0, 24), ((40, 40, 30), 0, 16),
    # the library's: rows of 96 to 1024 points only
    ((64, 64, 32), 0, 17), ((32, 128, 32), 0, 17), ((49, 49, 49), 0, 25),
    ((32, 32, 32), 1, 17), ((64, 64, 64), 1, 33), ((64, 128, 95), 1, 48), ((9, 10, 96), 1, 56),
    ((100, 100, 100), 1, 56), ((512, 512, 512), 1, 264), ((16, 1024, 1024), 1, 520),
    ((16, 1025, 1025), 1, 513), ((32, 2048, 2048), 1, 1025)])
def test_pitch(shape, walls, pitch):
    got = route([(shape, walls, 1)])[0]
    assert got[1] == pitch
    assert got[1] >= shape[2] // 2 + 1


def test_radices_multiply_to_the_length_and_the_twiddle_index_stays_in_range():
    lens = [n for n in range(2, 1100)]
    for p32 in (0, 1):
        got = route([((n, n, n), 0, p32) for n in lens])
        for n, (own, _, rad) in zip(lens, got):
            m = n
            for q in (2, 3, 5):
                while m % q == 0:
                    m //= q
            takes = m == 1 and n <= 1024
            assert bool(rad[0]) == takes and rad[0] == rad[1] == rad[2]
            if not takes:
                assert not own
                continue
            assert int(np.prod(rad[0])) == n and set(rad[0]) <= {2, 3, 4, 5, 6, 8}
            assert p32 or 6 not in rad[0]
            s = 1
            for R in rad[0]:
                step = n // (s * R)
                assert n % (s * R) == 0 and (s - 1) * (R - 1) * step < n
                # j div s by the multiplication of the kernel
                inv = ((1 << 20) + s - 1) // s
                j = np.arange(n // R, dtype=np.uint64)
                assert np.array_equal((j * inv) >> 20, j // s)
                s *= R


@pytest.mark.parametrize("shape,walls,own64,own32", [
    ((160, 180, 240), 0, True, True), ((32, 32, 32), 0, True, True), ((36, 64, 36), 0, True, True),
    ((100, 128, 30), 0, False, False),                                   # short rows, many lines
    ((128, 16, 128), 0, False, False), ((256, 16, 16), 0, False, False),  # small, powers of two
    ((256, 16, 256), 0, False, False), ((64, 8, 512), 0, False, False),
    ((256, 32, 256), 0, True, True), ((64, 64, 64), 0, True, True), ((120, 16, 128), 0, True, True),
    ((32, 16, 128), 0, True, True),
    ((28, 28, 28), 0, False, False), ((64, 64, 2048), 0, False, False),   # lengths it does not take
    ((256, 256, 256), 1, True, False), ((64, 128, 128), 1, False, False)])
def test_own_transforms_or_the_library(shape, walls, own64, own32):
    got = route([(shape, walls, p) for p in (0, 1)])
    assert [g[0] for g in got] == [own64, own32]
    if not walls and not got[0][0] and np.prod(shape) <= 1 << 20:
        assert all(g[1] == shape[2] // 2 + 1 for g in got)


def test_only_launched_shapes_of_columns_are_built():
    """Column kernels in double precision have tiles of eight columns: a tile of
    four is for single precision's lines of over 512 points."""
    lib = os.path.join(ROOT, "paper_2105_01865_amd", "libch.so")
    if not os.path.exists(lib):
        pytest.skip("libch.so not built")
    out = subprocess.run(["nm", "-C", lib], capture_output=True, text=True, check=True).stdout
    cols = [ln for ln in out.splitlines() if "k_fft_cols<" in ln or "k_fft_zsolve<" in ln]
    assert any("float, 4, 8, 512" in ln for ln in cols)
    assert not any("double, 4," in ln for ln in cols)


def test_the_gpu_test_s_shapes_reach_every_radix_and_launch_shape():
    from tests.test_gpu_fft_lines import LONG_Z, SHAPES
    for p32, radices in ((0, {2, 3, 4, 5, 8}), (1, {2, 3, 4, 5, 6, 8})):
        got = route([(s, 0, p32) for s in SHAPES + LONG_Z])
        own = [(s, g) for s, g in zip(SHAPES + LONG_Z, got) if g[0]]
        assert len(own) < len(got)          # and both sides of the rule
        for axis in range(3):
            assert set().union(*(g[2][axis] for _, g in own)) >= radices - {6}
            lens = [s[2 - axis] for s, _ in own]
            for lo, hi in ((1, 128), (128, 256), (256, 512), (512, 1024)):
                assert any(lo < n <= hi for n in lens), (axis, lo)
        assert any(6 in r for _, g in own for r in g[2]) == bool(p32)
