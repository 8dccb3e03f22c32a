"""The plan that a state reports, given back as options: the same bits (the
planner and the device code on the CPU, under AddressSanitizer and UBSan)."""
import os
import subprocess
import tempfile

import numpy as np
import pytest

from tests.harness_util import ROOT, run_emu
from tests.test_line_split import _box

_EXE = []


def reported(shapes, dt, prec=0, x_rows=0, z_chunk=0, seg_len=0, bc=(0, 0, 0)):
    """x_rows, z_chunk and seg_len as ch_autotune and ch_get_config report
    them for boxes (nz, ny, nx), and the longest segment of the plan."""
    if not _EXE:
        exe = os.path.join(tempfile.mkdtemp(prefix="ch_plan_"), "plan_dump")
        subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=undefined", "-fno-omit-frame-pointer", "-o", exe,
                        os.path.join(ROOT, "tests", "cpu_harness", "plan_dump.cpp")], check=True)
        _EXE.append(exe)
    text = f"{len(shapes)} {prec} {x_rows} {z_chunk} {seg_len} {dt!r}\n" + "".join(
        f"{nx} {ny} {nz} {1.0 / max(nz, ny, nx)!r} {bc[0]} {bc[1]} {bc[2]}\n"
        for nz, ny, nx in shapes)
    r = subprocess.run([_EXE[0]], input=text, capture_output=True, text=True,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0 and not r.stdout.startswith("FAIL"), r.stdout + r.stderr
    return dict(zip(("x_rows", "z_chunk", "seg_len", "longest"), map(int, r.stdout.split())))


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape,split", [((10, 281, 21), True), ((300, 24, 24), True),
                                         ((300, 30, 31), True), ((300, 300, 8), True),
                                         ((40, 300, 24), True), ((24, 24, 24), False)])
def test_the_reported_plan_gives_the_same_bits(shape, split, prec):
    b = _box(shape, (0, 0, 0), 4)
    t = reported([shape], 2e-4, prec)
    assert (t["longest"] < max(shape[:2])) == split
    auto, _, _ = run_emu([b], 2e-4, 1, prec=prec)
    again, _, plan = run_emu([b], 2e-4, 1, prec=prec, x_rows=t["x_rows"], z_chunk=t["z_chunk"],
                             seg=t["seg_len"])
    assert plan["seg"] == t["longest"]
    assert np.array_equal(again[0], auto[0])
