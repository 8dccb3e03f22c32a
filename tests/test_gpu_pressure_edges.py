"""The pressure solve where its kernels' blocks end: z extents around the
elimination's blocks of rows (8 in FP32, 4 in FP64) and around the mean
mode's chunks (1024 rows), padded and unpadded spectrum rows (from
nx/2 + 1 = 16 on), more than one wave of modes.

Bars as in test_gpu_pressure.py: FP64 1e-12 of the largest value, except
where the mean mode's two-term recurrence runs over more than 1000 rows,
whose error grows with nz^2 (nz^2 eps = 5e-10 at 1500 rows)."""
import numpy as np
import pytest
import torch

from oracle import pressure as pr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(7, 6, 28), (8, 6, 30), (9, 10, 31), (15, 6, 33), (16, 9, 32),
                                   (17, 6, 34), (18, 40, 62), (33, 5, 2)])
@pytest.mark.parametrize("zwalls", [False, True])
def test_solve_at_block_edges(shape, zwalls):
    from paper_2105_01865_amd import ch
    rng = np.random.default_rng([*shape, int(zwalls)])
    h = 1.0 / shape[2]
    rhs = rng.standard_normal(shape)
    ref = pr.poisson(rhs, h, zwalls)
    for prec, dt_, tol in (("fp64", torch.float64, 1e-12), ("fp32", torch.float32, 1e-5)):
        print(f"[gpu] poisson {shape} walls={zwalls} {prec}", flush=True)
        p = ch.Poisson(shape, h, z_walls=zwalls, precision=prec, stream=torch.cuda.Stream())
        x = torch.from_numpy(rhs).to("cuda", dt_)
        first = p.solve(x).double().cpu().numpy()
        again = p.solve(x).double().cpu().numpy()
        p.close()
        assert np.array_equal(first, again)
        assert np.abs(first - ref).max() / np.abs(ref).max() <= tol


@pytest.mark.parametrize("nz", [1023, 1024, 1025, 1500])
def test_mean_mode_across_chunks(nz):
    """A right-hand side that varies along z alone: only the mean mode."""
    from paper_2105_01865_amd import ch
    z = (np.arange(nz) + 0.5) / nz
    prof = np.cos(np.pi * z) + 0.3 * np.cos(7 * np.pi * z)
    h = 1.0 / nz
    # cosines are eigenvectors of the Neumann Laplacian
    lam = lambda k: -4.0 / h ** 2 * np.sin(0.5 * np.pi * k / nz) ** 2   # noqa: E731
    ref = np.cos(np.pi * z) / lam(1) + 0.3 * np.cos(7 * np.pi * z) / lam(7)
    rhs = np.broadcast_to(prof[:, None, None], (nz, 4, 6)).copy()
    print(f"[gpu] mean mode nz={nz}", flush=True)
    p = ch.Poisson((nz, 4, 6), h, z_walls=True, precision="fp64", stream=torch.cuda.Stream())
    got = p.solve(torch.from_numpy(rhs).cuda()).cpu().numpy()
    p.close()
    assert np.abs(got - ref[:, None, None]).max() / np.abs(ref).max() <= nz ** 2 * 2.3e-16
