"""A solve's start: one pass takes the velocity, the forces and f - G p from the
caller's arrays, whatever their row stride, and its end writes the velocity back.

With no iterations the velocity comes back bit for bit, and the residual norm is
that of stk_energy_norm of the same state: sums of n = nx ny terms of one sign
in another grouping, at most 64 roundings deep, and quotients of a few more, so
that 1e-13 relative is about 450 units of rounding."""
import numpy as np
import pytest
import torch

from paper_2509_19061_amd import inputs as I

pytestmark = pytest.mark.gpu


# tiles of 64 x 4: one, remainders of either side; strides other than the handle's
@pytest.mark.parametrize("nx,ny,align", [(16, 16, 64), (64, 48, 64), (68, 36, 128), (128, 132, 64), (128, 128, 256)])
@pytest.mark.parametrize("pressure", [False, True])
def test_no_iterations_give_back_the_start(nx, ny, align, pressure):
    from paper_2509_19061_amd import api, fields
    p = I.sinker_problem(nx, ny, [(0.4, 0.6, 0.1), (0.65, 0.35, 0.08)], 1e2, 1.0)
    ctx = api.Context(0)
    d = fields.DeviceProblem(p, torch.float64, align=align)
    m = api.MG(ctx, d.grid, d.eta_c, d.eta_n)
    vx0, vy0 = I.random_velocity(p, 21, 1e-3)
    vx, vy = d.velocity(vx0, vy0)
    pt = d.field(np.random.default_rng(nx).standard_normal((ny, nx))) if pressure else None
    norm = api.energy_norm(ctx, "f64", d.grid, vx, vy, pt, d.eta_c, d.eta_n, d.fx, d.fy)
    rep = m.solve("f64", vx, vy, pt, d.fx, d.fy, tol=1e-100, max_iters=0, allow_notconv=True)
    torch.cuda.synchronize()
    assert np.array_equal(d.get_vx(vx), vx0) and np.array_equal(d.get_vy(vy), vy0)
    assert rep["iterations"] == 0
    assert abs(rep["ev"] - norm[4]) <= 1e-13 * norm[4]
    m.close()
    ctx.close()
