"""Lines of a small box split at the ends of their chunks (the automatic plan
of a single box with few y or z lines): the same bits as whole lines, on the
CPU under AddressSanitizer and UBSan, periodic and between walls, in every
solve precision; the oracle's step; and a box that is not split."""
import numpy as np
import pytest

import oracle
from paper_2105_01865_amd import inputs
from tests.harness_util import run_emu


def _box(shape, bc, seed):
    rng = np.random.default_rng(seed)
    h = 1.0 / max(shape)
    C = 0.5 + 0.3 * rng.normal(size=shape)
    u, v, w = inputs.wall_velocity(rng, shape, bc, h)
    s = 1.0 / max(np.abs(u).max(), np.abs(v).max(), np.abs(w).max())
    return dict(C=C, u=u * s, v=v * s, w=w * s, h=h, Cn=h, Pe=0.9 / h, bc=bc)


@pytest.mark.parametrize("prec,solve", [(0, 0), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape,bc", [
    ((8, 300, 9), (0, 0, 0)),     # 38-point chunks: eight, the last one shorter
    ((8, 210, 33), (0, 1, 0)),    # walls at both ends of the line; 32 + 1 columns
    ((257, 8, 8), (0, 0, 1)),     # z lines, ragged last segment
    ((300, 9, 10), (1, 0, 0)),
])
def test_split_lines_give_the_bits_of_whole_lines(shape, bc, prec, solve):
    b = _box(shape, bc, 3)
    dt = 2e-4
    n = max(shape)
    split, ms, ps = run_emu([b], dt, 2, prec=prec, solve=solve)
    whole, mw, pw = run_emu([b], dt, 2, prec=prec, solve=solve, seg=n)
    assert ps["seg"] < n and pw["seg"] == n
    assert np.array_equal(split[0], whole[0]) and ms == mw
    ref = oracle.step(b["C"], b["u"], b["v"], b["w"], b["h"], b["Cn"], b["Pe"], dt, 2, bc=bc)
    assert np.abs(split[0] - ref).max() / np.abs(ref).max() < (1e-12 if prec == 0 else 2e-6)


def test_a_box_in_a_batch_has_the_bits_of_the_box_alone():
    shapes = [(8, 200, 10), (10, 9, 12)]
    boxes = [_box(s, (0, 0, 0), 5 + i) for i, s in enumerate(shapes)]
    got, _, _ = run_emu(boxes, 2e-4, 1)
    for b, g in zip(boxes, got):
        (alone,), _, _ = run_emu([b], 2e-4, 1)
        assert np.array_equal(g, alone)


def test_short_lines_stay_whole():
    b = _box((24, 24, 24), (0, 0, 0), 9)
    _, _, plan = run_emu([b], 1e-4, 1)
    assert plan["seg"] == 24
