"""RAS outer iterations with a thin overlap on the register pipeline, against the
kernel that keeps each tile's window in LDS (bit for bit) and the CPU oracle.

Tiles of one strip and of several (64 columns hold a tile of up to 62 - 2 h), clipped
tiles at every side, tiles larger than the grid, several segments of a tile's rows,
overlaps from none to k - 2, and sweep counts up to the largest of a pass.  Oracle
bars: FP64 normwise 1e-12, FP32 1e-5 per sweep.
"""
import os

import pytest
import torch

from gpu_util import as_dtype, normwise
from oracle import stokes as S
from paper_2509_19061_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctxs():
    from paper_2509_19061_amd import api
    auto = api.Context(0)
    os.environ["STK_RAS_KERNEL"] = "window"
    try:
        window = api.Context(0)
    finally:
        del os.environ["STK_RAS_KERNEL"]
    yield auto, window
    auto.close()
    window.close()


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nx,ny", [(61, 47), (130, 200), (201, 66)])
@pytest.mark.parametrize("tx,ty,h,k,sx,sy", [(64, 64, 0, 2, 0, 0), (64, 64, 0, 4, 17, 63), (32, 32, 0, 8, 5, 1),
                                             (62, 20, 0, 3, 61, 19), (60, 30, 1, 4, 1, 2), (63, 48, 0, 7, 40, 3),
                                             (8, 9, 2, 5, 3, 8), (100, 80, 3, 6, 99, 0), (300, 40, 0, 4, 0, 15),
                                             (64, 16, 4, 10, 9, 15), (24, 64, 0, 9, 23, 30)])
def test_thin_overlap_equals_the_window_kernel_and_the_oracle(ctxs, nx, ny, tx, ty, h, k, sx, sy, dtype):
    from paper_2509_19061_amd import api, fields
    p = I.sinker_problem(nx, ny, [(0.3, 0.4, 0.2), (0.7, 0.6, 0.15)], 1e4, 1.0)
    for f in ("eta_c", "eta_n", "fx", "fy"):
        setattr(p, f, as_dtype(getattr(p, f), dtype))
    vx0, vy0 = (as_dtype(v, dtype) for v in I.random_velocity(p, nx + ny, 1e-2))
    dp = fields.DeviceProblem(p, dtype)
    vx, vy = dp.velocity(vx0, vy0)
    out = []
    for c in ctxs:
        gx, gy = dp.field() + 7, dp.field() + 7
        api.ras_outer(c, dtype, dp.grid, vx, vy, dp.eta_c, dp.eta_n, dp.fx, dp.fy, gx, gy, 0.7, tx, ty, h, k, sx, sy)
        out.append((gx, gy))
    assert torch.equal(out[0][0][:ny, :nx + 1], out[1][0][:ny, :nx + 1])
    assert torch.equal(out[0][1][:ny + 1, :nx], out[1][1][:ny + 1, :nx])
    bx, by = S.rhs(p, p.fx, p.fy)
    ox, oy = S.ras_outer(p, bx, by, 0.7, tx, ty, h, k, sx, sy, vx0, vy0)
    tol = 1e-12 if dtype == torch.float64 else k * 1e-5
    assert normwise(dp.get_vx(out[0][0]), ox) <= tol and normwise(dp.get_vy(out[0][1]), oy) <= tol
    # nothing outside the used extents is written
    gx, gy = out[0]
    assert bool((gx[ny:] == 7).all()) and bool((gx[:, nx + 1:] == 7).all()) and bool((gy[:, nx:] == 7).all())


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_non_finite_values_stay_in_the_windows_that_hold_them(ctxs, dtype):
    """Eight sweeps, cuts every 24 columns and 21 rows: what a tile does not see stays finite."""
    from paper_2509_19061_amd import api, fields
    p = I.sinker_problem(90, 70, [(0.3, 0.4, 0.2)], 1e2, 1.0)
    dp = fields.DeviceProblem(p, dtype)
    for h in (0, 1):
        vx, vy = dp.velocity(*I.random_velocity(p, 5, 1e-2))
        vx[22, 40], vy[43, 26], vx[19, 70], vy[63, 79] = float("nan"), float("inf"), -float("inf"), float("nan")
        out = []
        for c in ctxs:
            gx, gy = dp.field(), dp.field()
            api.ras_outer(c, dtype, dp.grid, vx, vy, dp.eta_c, dp.eta_n, dp.fx, dp.fy, gx, gy, 0.7, 24, 21, h, 8, 0, 0)
            out.append((gx, gy))
        for a, b in zip(*out):
            assert torch.equal(a.isnan(), b.isnan()) and bool(a.isnan().any()) and bool(a.isfinite().any())
            assert torch.equal(a.nan_to_num(7.0), b.nan_to_num(7.0))
