"""The pressure solve's own transforms: every radix (2, 3, 4, 5, 6, 8) and their
mixtures along each axis, the edges of the tiles of columns and rows, of the
launch shapes (64, 128, 256, 512 and 1024 points), extents that are no product of
2, 3 and 5, and both sides of the rule that leaves a mesh to the FFT library.

Bars as in test_gpu_pressure.py (of the largest value): FP64 1e-12, FP32 1e-5
(the transforms' own error is a few eps times log2 n).  With walls the
elimination's rounded diagonal 2 + lambda h^2 adds eps n^2 / 2 pi^2 at lines of n
points along x or y, and the mean mode nz^2 eps."""
import numpy as np
import pytest
import torch

from oracle import pressure as pr

pytestmark = pytest.mark.gpu

SHAPES = [(2, 3, 4), (5, 8, 9), (10, 12, 15), (27, 25, 16), (20, 18, 30), (6, 40, 32), (9, 64, 60),
          (16, 15, 34), (30, 14, 32), (11, 16, 18), (4, 6, 256), (3, 5, 270), (2, 4, 512),
          (3, 2, 540), (2, 3, 1024), (2, 3, 1030), (3, 256, 36), (2, 288, 40), (3, 512, 45),
          (2, 600, 48), (3, 1024, 50), (8, 128, 64), (8, 125, 65), (60, 64, 35), (60, 64, 36)]
LONG_Z = [(256, 6, 9), (300, 5, 10), (512, 4, 18), (640, 3, 16), (1000, 2, 15), (1024, 3, 8)]


@pytest.mark.parametrize("shape", SHAPES + LONG_Z)
def test_periodic(shape):
    from paper_2105_01865_amd import ch
    rng = np.random.default_rng(shape)
    h = 1.0 / max(shape)
    rhs = rng.standard_normal(shape)
    ref = pr.poisson(rhs, h, False)
    for prec, dt_, tol in (("fp64", torch.float64, 1e-12), ("fp32", torch.float32, 1e-5)):
        print(f"[gpu] poisson {shape} {prec}", flush=True)
        p = ch.Poisson(shape, h, z_walls=False, precision=prec, stream=torch.cuda.Stream())
        got = p.solve(torch.from_numpy(rhs).to("cuda", dt_)).double().cpu().numpy()
        p.close()
        assert np.abs(got - ref).max() / np.abs(ref).max() <= tol


@pytest.mark.parametrize("shape", [(63, 256, 256), (64, 256, 256), (65, 256, 257), (50, 300, 300),
                                   (17, 512, 512), (5, 1000, 1000), (3, 240, 180)])
def test_walls(shape):
    from paper_2105_01865_amd import ch
    rng = np.random.default_rng(shape)
    h = 1.0 / max(shape)
    rhs = rng.standard_normal(shape)
    ref = pr.poisson(rhs, h, True)
    eps = np.finfo(float).eps
    print(f"[gpu] poisson {shape} walls fp64", flush=True)
    p = ch.Poisson(shape, h, z_walls=True, precision="fp64", stream=torch.cuda.Stream())
    got = p.solve(torch.from_numpy(rhs).cuda()).cpu().numpy()
    p.close()
    tol = 1e-12 + eps * (max(shape) ** 2 / (2 * np.pi ** 2) + shape[0] ** 2)
    assert np.abs(got - ref).max() / np.abs(ref).max() <= tol
