"""3D residual and norm on grids large enough for the plane walk (more than three gathering
workgroups per CU, 64 x 4 columns of one plane each) and just below, against the CPU
oracle; ragged in every direction, with segments that do not divide the planes.

Bars: FP64 normwise 1e-12 (norms: relative 1e-11); FP32 1e-5 (norms 1e-4).
"""
import numpy as np
import pytest
import torch

from gpu_util import as_dtype, normwise
from oracle import stokes3d as S3
from paper_2509_19061_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("dims", [(7, 5, 385), (9, 2, 769), (70, 66, 23), (129, 65, 30), (47, 47, 47), (3, 1030, 3)])
def test_residual_and_norm_match_oracle(dims, dtype):
    from paper_2509_19061_amd import api, fields
    ctx = api.Context(0)
    p = I.sinker_problem3d(*dims, [(0.4, 0.6, 0.5, 0.25)], 1e3, 1.0)
    p = I.Problem3(p.nx, p.ny, p.nz, p.dx, p.dy, p.dz,
                   *(as_dtype(a, dtype) for a in (p.eta_c, p.eta_xy, p.eta_xz, p.eta_yz, p.fx, p.fy, p.fz)))
    v0 = tuple(as_dtype(a, dtype) for a in I.random_velocity3d(p, 3, 1e-3))
    d = fields.DeviceProblem3(p, dtype)
    v, r = d.velocity(v0), d.velocity()
    api.residual3d(ctx, dtype, d.grid, v, d.eta, d.f, r)
    e = api.energy_norm3d(ctx, dtype, d.grid, v, d.eta, d.f)
    torch.cuda.synchronize()
    for got, ref in zip(d.get_v(r), S3.residual(p, *v0, p.fx, p.fy, p.fz)):
        assert normwise(got, ref) <= (1e-12 if dtype == torch.float64 else 1e-5)
    np.testing.assert_allclose(np.asarray(e)[:2], np.asarray(S3.energy(p, *v0, p.fx, p.fy, p.fz))[:2],
                               rtol=1e-11 if dtype == torch.float64 else 1e-4)
    ctx.close()
