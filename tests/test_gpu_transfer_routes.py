"""Coarse-to-fine transfers on both sides of the rules that choose the kernel
where the taps are selected (ch_route.h): enough groups for the marching kernel
in each of its forms, with ragged rows and planes, and shapes that stay with the
general kernel, its piped form among them.  Bars as in test_gpu_multires.py:
FP64 1e-13 and FP32 2e-6 of the largest velocity."""
import numpy as np
import pytest

import oracle
from paper_2105_01865_amd import inputs
from tests.test_transfer_route import routes


@pytest.mark.gpu
@pytest.mark.parametrize("fine,nc,march", [
    ((770, 24, 60), (130, 8, 20), (True, True)),       # ratio 3, four sub-bands
    ((402, 31, 150), (150, 20, 96), (True, True)),     # ratio 1.5, two
    ((262, 25, 387), (100, 8, 129), (True, True)),     # ratio 3, one
    ((402, 25, 211), (100, 16, 132), (True, True)),    # 11 rows, odd target rows
    ((262, 24, 208), (100, 15, 130), (True, False)),   # 11 rows, rows of 4 targets
    ((50, 15, 320), (40, 12, 256), (False, False)),    # FP32: piped
    ((12, 230, 230), (12, 230, 230), (False, False)),  # ratio 1, piped
    ((32, 120, 120), (24, 48, 48), (False, False)),
])
def test_both_sides_of_the_rule_match_the_oracle(fine, nc, march):
    import torch
    from paper_2105_01865_amd import ch
    nz, ny, nx = fine
    rng = np.random.default_rng([*fine, *nc])
    zf = inputs.stretched_faces(nc[0], 2.0)
    uc, vc, wc = (rng.standard_normal((nc[0] + (d == 2), nc[1], nc[2])) for d in range(3))
    wc[0] = wc[-1] = 0.0
    ref = oracle.interp_velocity(zf, uc, vc, wc, (nx, ny, nz))
    for prec, dt_, tol, es, m in (("fp64", torch.float64, 1e-13, 8, march[1]),
                                  ("fp32", torch.float32, 2e-6, 4, march[0])):
        (r,) = routes([(nc, fine, es, 16)])
        assert r[0][1] == m   # u
        print(f"[gpu] transfer routes fine={fine} coarse={nc} {prec}", flush=True)
        ip = ch.Interp(fine, 1.0 / nx, nc, zf, precision=prec, stream=torch.cuda.Stream())
        c = [torch.from_numpy(a).to("cuda", dt_) for a in (uc, vc, wc)]
        out = tuple(torch.full(s, 7.0, dtype=dt_, device="cuda")
                    for s in ((nz, ny, nx), (nz, ny, nx), (nz + 1, ny, nx)))
        got = ip.apply(*c, out=out)
        torch.cuda.synchronize()
        for g, want in zip(got, ref):
            assert np.abs(g.double().cpu().numpy() - want).max() <= tol * np.abs(want).max()
        ip.close()
