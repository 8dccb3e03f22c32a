"""The explicit 25-point scheme's row program (one x-line per task, the y
stencil in registers, the rows at two planes alternating in LDS).

On the CPU (the kernel's own code under AddressSanitizer and UBSan, the
library's plan and LDS size): the same bits as the general program on every
boundary combination, ragged extents and march lengths, and the oracle's
scheme.  On the GPU: against the oracle at work-group edges."""
import os
import subprocess
import tempfile

import numpy as np
import pytest

import oracle
from paper_2105_01865_amd import inputs
from tests.harness_util import ROOT, pack

_EXE = []


def _exe():
    if not _EXE:
        exe = os.path.join(tempfile.mkdtemp(prefix="ch_e25_"), "emu_e25")
        subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=undefined", "-fno-omit-frame-pointer", "-o", exe,
                        os.path.join(ROOT, "tests", "cpu_harness", "emu_e25.cpp")], check=True)
        _EXE.append(exe)
    return _EXE[0]


def _box(shape, bc, seed):
    rng = np.random.default_rng(seed)
    h = 1.0 / max(shape)
    C = 0.5 + 0.3 * rng.normal(size=shape)
    u, v, w = inputs.wall_velocity(rng, shape, bc, h)
    s = 1.0 / max(np.abs(u).max(), np.abs(v).max(), np.abs(w).max())
    return dict(C=C, u=u * s, v=v * s, w=w * s, h=h)


def _ref(b, dt, bc, steps):
    return oracle.step_explicit25(b["C"], b["u"], b["v"], b["w"], b["h"], b["h"], 0.9 / b["h"], dt,
                                  steps, bc=bc)


CASES = [((10, 9, 8), (0, 0, 0), 3), ((7 + 1, 10, 17), (1, 0, 0), 1), ((9, 13, 16), (0, 1, 0), 4),
         ((12, 8, 64), (0, 0, 1), 5), ((11, 10, 65), (1, 1, 1), 2), ((9, 1, 24), (0, 0, 0), 9),
         ((1, 12, 20), (0, 0, 0), 1), ((20, 8, 33), (1, 0, 1), 0), ((8, 9, 70), (0, 0, 0), 8)]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape,bc,zc", CASES)
def test_same_bits_as_the_general_program(shape, bc, zc, prec):
    b = _box(shape, bc, 5)
    h = b["h"]
    dt = 0.3 * 2.5 * 0.9 * h / 144.0
    nz, ny, nx = shape
    with tempfile.TemporaryDirectory() as d:
        with open(os.path.join(d, "params.txt"), "w") as f:
            f.write(f"1 {prec} 4.0 1e-6 0 0 0 0 {zc} {dt!r} 2 1 0\n{nx} {ny} {nz} {h!r} {h!r} "
                    f"{0.9 / h!r} {bc[0]} {bc[1]} {bc[2]}\n")
        for name in ("C", "u", "v", "w"):
            pack([b[name]]).tofile(os.path.join(d, name + ".bin"))
        env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=1",
                   UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1")
        r = subprocess.run([_exe(), os.path.join(d, "params.txt"), d, d], env=env,
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
        general = np.fromfile(os.path.join(d, "C.bin")).reshape(shape)
        row = np.fromfile(os.path.join(d, "C_row.bin")).reshape(shape)
    assert np.array_equal(row, general)
    assert np.array_equal(row, general)
    ref = _ref(b, dt, bc, 2)
    assert np.abs(row - ref).max() / np.abs(ref).max() < (1e-12 if prec == 0 else 2e-6)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,bc", [((11, 9, 63), (0, 0, 0)), ((20, 10, 64), (1, 0, 1)),
                                      ((17, 12, 257), (0, 1, 0)), ((9, 8, 512), (0, 0, 0)),
                                      ((8, 9, 1000), (1, 1, 1))])
def test_gpu_matches_oracle(shape, bc):
    """FP64 1e-12 and FP32 5e-6 of the largest value, the parity bars of the
    explicit scheme; the plan reports the row program."""
    import torch
    from paper_2105_01865_amd import ch
    b = _box(shape, bc, 6)
    h = b["h"]
    dt = 0.3 * 2.5 * 0.9 * h / 144.0
    ref = _ref(b, dt, bc, 2)
    for prec, dt_, tol in (("fp64", torch.float64, 1e-12), ("fp32", torch.float32, 5e-6)):
        print(f"[gpu] explicit row {shape} bc={bc} {prec}", flush=True)
        s = ch.State(shape, h, h, 0.9 / h, bc=bc, precision=prec, stream=torch.cuda.Stream())
        C, u, v, w = (torch.from_numpy(b[k]).to("cuda", dt_).contiguous() for k in "Cuvw")
        s.set_field(C)
        s.step_explicit25(u, v, w, dt, 2)
        got = s.get_field().double().cpu().numpy()
        assert s.x_program() == 1
        s.close()
        assert np.abs(got - ref).max() / np.abs(ref).max() <= tol
