"""Drops of boxes with axes of one cell: the labelling folds such axes away, on
the CPU the rule, on the GPU (root, cells) lists equal to the flood fill's."""
import itertools
import os
import subprocess
import tempfile

import numpy as np
import pytest

import oracle
from tests.harness_util import ROOT


def test_folded_box_keeps_indices_and_boundaries():
    cases = [(n, b) for n in itertools.product((1, 8, 13), repeat=3)
             for b in ((0, 0, 0), (1, 0, 1), (0, 1, 0), (1, 1, 1))]
    exe = os.path.join(tempfile.mkdtemp(prefix="ch_axes_"), "axes_dump")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=undefined", "-o", exe,
                    os.path.join(ROOT, "tests", "cpu_harness", "axes_dump.cpp")], check=True)
    r = subprocess.run([exe], input="".join(" ".join(map(str, (*n, *b))) + "\n" for n, b in cases),
                       capture_output=True, text=True, check=True,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    for (n, b), line in zip(cases, r.stdout.splitlines()):
        v = list(map(int, line.split()))
        kept = [(q, c) for q, c in zip(n, b) if q > 1]
        got = list(zip(v[:3], v[3:]))
        # the axes of more than one cell in their order, so that x + nx (y + ny z)
        # is the same number; the others join nothing
        assert got[:len(kept)] == kept
        assert all(q == (1, 1) for q in got[len(kept):])


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(3001, 1, 1), (1, 3001, 1), (1, 1, 3001), (130, 70, 1),
                                   (130, 1, 70), (1, 130, 70), (1, 1, 1)])
@pytest.mark.parametrize("p", [0.3, 0.9, 1.0])
def test_gpu_matches_flood_fill(shape, p):
    import torch
    from paper_2105_01865_amd import ch
    C = (np.random.default_rng([*shape, int(10 * p)]).random(shape) < p).astype(np.float64)
    for bc in ((0, 0, 0), (1, 1, 1)):
        print(f"[gpu] drops {shape} p={p} bc={bc}", flush=True)
        s = ch.State(shape, 0.01, 0.01, 90.0, bc=bc, precision="fp64", stream=torch.cuda.Stream())
        s.set_field(torch.from_numpy(C).to("cuda"))
        got = [s.drops(0.5) for _ in range(2)]
        s.close()
        lab, nd = oracle.label_drops(C, 0.5, bc=bc)
        roots, cells, _, _ = oracle.drop_volumes(lab, 1.0)
        for r, c in got:
            assert len(r) == nd and np.array_equal(r, roots) and np.array_equal(c, cells)
