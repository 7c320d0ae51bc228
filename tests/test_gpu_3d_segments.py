"""The 3D plane walk cut into segments of equal planes (2 to 32 of them, as many
segments as fill the chip), against the CPU oracle: sweeps, residual and norm on grids
whose last segment is shorter, whose planes do not fill one, and with one tile or many.

Bars: FP64 normwise 1e-12 (norms: relative 1e-11); FP32 1e-5 per sweep from the same
state rounded to FP32.
"""
import numpy as np
import pytest
import torch

from gpu_util import as_dtype, normwise
from oracle import stokes3d as S3
from paper_2509_19061_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("dims", [(2, 2, 2), (5, 6, 3), (9, 5, 7), (65, 5, 13), (12, 9, 37), (7, 6, 129), (130, 70, 35)])
def test_segments_match_oracle(dims, dtype):
    from paper_2509_19061_amd import api, fields
    ctx = api.Context(0)
    p = I.sinker_problem3d(*dims, [(0.4, 0.6, 0.5, 0.25)], 1e3, 1.0)
    p = I.Problem3(p.nx, p.ny, p.nz, p.dx, p.dy, p.dz,
                   *(as_dtype(a, dtype) for a in (p.eta_c, p.eta_xy, p.eta_xz, p.eta_yz, p.fx, p.fy, p.fz)))
    v0 = tuple(as_dtype(a, dtype) for a in I.random_velocity3d(p, 3, 1e-3))
    dp = fields.DeviceProblem3(p, dtype)
    v, r = dp.velocity(v0), dp.velocity()
    api.residual3d(ctx, dtype, dp.grid, v, dp.eta, dp.f, r)
    e = api.energy_norm3d(ctx, dtype, dp.grid, v, dp.eta, dp.f)
    api.smooth3d(ctx, dtype, dp.grid, v, dp.eta, dp.f, 1, "jacobi_fused")
    torch.cuda.synchronize()
    tol = 1e-12 if dtype == torch.float64 else 1e-5
    for got, ref in ((dp.get_v(r), S3.residual(p, *v0, p.fx, p.fy, p.fz)),
                     (dp.get_v(v), S3.jacobi(p, p.fx, p.fy, p.fz, 0.7, *v0))):
        for g, o in zip(got, ref):
            assert normwise(g, o) <= tol
    np.testing.assert_allclose(np.asarray(e)[:2], np.asarray(S3.energy(p, *v0, p.fx, p.fy, p.fz))[:2],
                               rtol=1e-11 if dtype == torch.float64 else 1e-4)
    ctx.close()
