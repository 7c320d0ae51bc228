"""RAS outer iterations on grids of a few tiles, where the kernels that keep a tile in LDS
are faster than a pipelined pass and take over: thin and full overlap, both sides of the
line, against the CPU oracle.

Bars: FP64 normwise 1e-12, FP32 1e-5 per sweep from the same state rounded to FP32.
"""
import pytest
import torch

from gpu_util import as_dtype, normwise
from oracle import stokes as S
from paper_2509_19061_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nx,ny", [(2, 2), (4, 4), (16, 17), (33, 20), (200, 3), (3, 90), (150, 140)])
def test_outer_iterations_match_oracle(nx, ny, dtype):
    from paper_2509_19061_amd import api, fields
    ctx = api.Context(0)
    p = I.sinker_problem(nx, ny, [(0.3, 0.4, 0.2), (0.7, 0.6, 0.15)], 1e4, 1.0)
    for f in ("eta_c", "eta_n", "fx", "fy"):
        setattr(p, f, as_dtype(getattr(p, f), dtype))
    vx0, vy0 = (as_dtype(v, dtype) for v in I.random_velocity(p, nx + ny, 1e-2))
    dp = fields.DeviceProblem(p, dtype)
    vx, vy = dp.velocity(vx0, vy0)
    gx, gy = dp.velocity()
    bx, by = S.rhs(p, p.fx, p.fy)
    for tile, h, k in ((32, 0, 8), (16, 3, 10), (8, 1, 6), (64, 7, 8), (8, 10, 10), (16, 6, 7), (32, 0, 4)):
        api.ras_outer(ctx, dtype, dp.grid, vx, vy, dp.eta_c, dp.eta_n, dp.fx, dp.fy, gx, gy, 0.7, tile, tile, h, k,
                      3, 5)
        torch.cuda.synchronize()
        ox, oy = S.ras_outer(p, bx, by, 0.7, tile, tile, h, k, 3, 5, vx0, vy0)
        tol = 1e-12 if dtype == torch.float64 else k * 1e-5
        assert normwise(dp.get_vx(gx), ox) <= tol and normwise(dp.get_vy(gy), oy) <= tol, (tile, h, k)
    ctx.close()
