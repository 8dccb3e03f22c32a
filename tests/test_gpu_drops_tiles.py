"""The tiled drop labelling at the sizes where a tile (64 x 8 x 8 cells, one
row per wave) can go wrong: whole and ragged tiles, one tile whose axis wraps
onto itself, runs that cross every tile face, drops that pass through a tile
several times, and more tile roots than the first list holds.

Bar: (root, cells) lists are integers and must equal the flood fill's."""
import numpy as np
import pytest
import torch

import oracle
from paper_2105_01865_amd import ch

pytestmark = pytest.mark.gpu


def _check(C, bc, prec):
    dt_ = torch.float64 if prec == "fp64" else torch.float32
    h = 1.0 / C.shape[2]
    s = ch.State(C.shape, h, h, 0.9 / h, bc=bc, precision=prec, stream=torch.cuda.Stream())
    s.set_field(torch.from_numpy(np.ascontiguousarray(C)).to("cuda", dt_))
    first = s.drops(0.5)
    again = s.drops(0.5)
    s.close()
    Cp = C if prec == "fp64" else C.astype(np.float32).astype(np.float64)
    lab, nd = oracle.label_drops(Cp, 0.5, bc=bc)
    roots, cells, _, _ = oracle.drop_volumes(lab, 1.0)
    for r, c in (first, again):
        assert len(r) == nd
        assert np.array_equal(r, roots) and np.array_equal(c, cells)


@pytest.mark.parametrize("shape", [(8, 8, 64), (9, 17, 65), (16, 16, 128), (8, 10, 63),
                                   (24, 8, 130), (17, 33, 191), (1, 20, 70), (12, 1, 129),
                                   (10, 9, 1)])
@pytest.mark.parametrize("p", [0.1, 0.33, 0.7])
def test_tile_edges_match_flood_fill(shape, p):
    rng = np.random.default_rng([*shape, int(100 * p)])
    C = (rng.random(shape) < p).astype(np.float64)
    for bc in ((0, 0, 0), (1, 0, 1), (0, 1, 0), (1, 1, 1)):
        print(f"[gpu] drops {shape} p={p} bc={bc}", flush=True)
        _check(C, bc, "fp32" if bc[0] else "fp64")


def test_lines_through_every_tile_face():
    """A comb: parallel lines joined at one end only, along each axis."""
    shape = (33, 26, 150)
    for axis in range(3):
        C = np.zeros(shape)
        sel = [slice(None, None, 2)] * 3
        sel[axis] = slice(None)
        C[tuple(sel)] = 1.0
        sel = [slice(None)] * 3
        sel[axis] = 0
        C[tuple(sel)] = 1.0
        print(f"[gpu] drops comb along axis {axis}", flush=True)
        _check(C, (1, 1, 1), "fp64")
        _check(C, (0, 0, 0), "fp32")


def test_more_roots_than_the_first_list_holds():
    # isolated cells: half of the box's cells are drops of their own
    C = np.indices((40, 48, 64)).sum(0) % 2 * 1.0
    print("[gpu] drops checkerboard", flush=True)
    _check(C, (0, 0, 0), "fp64")
    rng = np.random.default_rng(7)
    _check(rng.random((40, 64, 96)), (0, 0, 1), "fp32")
