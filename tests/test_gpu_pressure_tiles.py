"""The pressure step's cell kernels where their tiles change: rows around
multiples of 64, 128 and 256 columns, few and many rows and planes (marches of
4, 8 and 16 planes), against the oracle's step.

Bars, of the largest value of each field: those of test_gpu_pressure.py (FP64
1e-12, FP32 5e-6); the velocity takes P's difference over a cell, and P is up to
n / 2 pi cells' differences large, so its rounding adds 4 eps n / 2 pi on lines of
n; between walls the elimination along z adds eps (n^2 / 2 pi^2 + nz^2)."""
import numpy as np
import pytest
import torch

from oracle import pressure as pr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(3, 5, 64), (9, 6, 65), (17, 3, 128), (5, 9, 129), (16, 5, 192),
                                   (33, 4, 255), (6, 7, 256), (4, 3, 257), (5, 2, 384), (8, 70, 20),
                                   (65, 40, 36), (40, 130, 130)])
@pytest.mark.parametrize("zwalls", [False, True])
def test_step_at_tile_edges(shape, zwalls):
    from paper_2105_01865_amd import ch
    nz, ny, nx = shape
    rng = np.random.default_rng([*shape, int(zwalls)])
    h = 1.0 / nx
    f = [rng.uniform(-0.1, 1.1, shape)] + [rng.standard_normal(shape) for _ in range(5)]
    if zwalls:
        f[3] = rng.standard_normal((nz + 1, ny, nx))
        f[3][0] = f[3][-1] = 0.0
    ref = pr.pressure_step(*f, h, 1e-3, 1000.0, 1.0, zwalls)
    for prec, dt_, base in (("fp64", torch.float64, 1e-12), ("fp32", torch.float32, 5e-6)):
        print(f"[gpu] pressure step {shape} walls={zwalls} {prec}", flush=True)
        eps, n = torch.finfo(dt_).eps, max(shape)
        tol = base + eps * 4 * n / (2 * np.pi)
        if zwalls:
            tol += eps * (n ** 2 / (2 * np.pi ** 2) + nz ** 2)
        p = ch.Poisson(shape, h, z_walls=zwalls, precision=prec, stream=torch.cuda.Stream())
        T = [torch.from_numpy(a).to("cuda", dt_) for a in f]
        p.step(*T, 1000.0, 1.0, 1e-3)
        torch.cuda.synchronize()
        p.close()
        for name, t, r in zip(("u", "v", "w", "P"), T[1:5], ref[:4]):
            e = np.abs(t.double().cpu().numpy() - r).max() / np.abs(r).max()
            print(f"  {name}: rel {e:.2e}")
            assert e <= tol
