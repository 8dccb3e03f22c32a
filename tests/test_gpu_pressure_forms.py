"""The tridiagonal solve along z on both sides of the row counts where its form
changes (32 in FP64, 192 in FP32), on planes of one wave of modes and of many, and
the same right-hand side in planes of few rows.

The right-hand side has no mean in any plane, so that the mean mode, whose
rounding grows with nz^2, stays out; bars as in test_gpu_pressure.py (FP64 1e-12,
FP32 1e-5 of the largest value) and eps n^2 / 2 pi^2 of the elimination's rounded
diagonal at lines of n points along x or y."""
import numpy as np
import pytest
import torch

from oracle import pressure as pr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(30, 6, 8), (31, 7, 9), (32, 6, 8), (33, 5, 12), (32, 40, 34),
                                   (190, 6, 8), (191, 4, 9), (192, 6, 8), (193, 5, 10),
                                   (2, 130, 150), (3, 128, 128), (8, 200, 96), (17, 100, 130)])
def test_forms_of_the_solve_along_z(shape):
    from paper_2105_01865_amd import ch
    rng = np.random.default_rng(shape)
    h = 1.0 / max(shape)
    rhs = rng.standard_normal(shape)
    rhs -= rhs.mean(axis=(1, 2), keepdims=True)
    ref = pr.poisson(rhs, h, True)
    n = max(shape[1:])
    for prec, dt_, tol, eps in (("fp64", torch.float64, 1e-12, 2.3e-16),
                                ("fp32", torch.float32, 1e-5, 1.2e-7)):
        print(f"[gpu] poisson forms {shape} {prec}", flush=True)
        x = torch.from_numpy(rhs).to("cuda", dt_)
        x -= x.mean(dim=(1, 2), keepdim=True)
        p = ch.Poisson(shape, h, z_walls=True, precision=prec, stream=torch.cuda.Stream())
        got = p.solve(x).double().cpu().numpy()
        p.close()
        got -= got.mean(axis=(1, 2), keepdims=True)
        assert np.abs(got - ref).max() / np.abs(ref).max() <= tol + eps * n ** 2 / (2 * np.pi ** 2)
