"""The pressure step where its passes change: the mean formed by the pass that
removes it up to 1024 workgroups of 64 x 32 cells, by a launch of its own
beyond; ragged rows and columns of a lane's eight rows.

Tolerance: the update is a few roundings per cell and the mean the rounding of
a sum in chunks of 8 rows, 64 lanes, 4 waves and at most 32 partials a lane, so
that 1e-13 normwise is 450 units of rounding."""
import numpy as np
import pytest
import torch

from gpu_util import normwise
from oracle import uzawa as U
from paper_2509_19061_amd import inputs as I

pytestmark = pytest.mark.gpu


# one cell row and more; 1, 2, 1024 (the last with the mean inside) and 1056 workgroups
@pytest.mark.parametrize("nx,ny", [(2, 2), (64, 32), (65, 33), (63, 7), (129, 41), (2048, 1024), (2047, 1017),
                                   (2049, 1024)])
def test_pressure_step_and_mean_match_oracle(nx, ny):
    from paper_2509_19061_amd import api, fields
    p = I.sinker_problem(nx, ny, [(0.4, 0.6, 0.2)], 1e3, 1.0)
    ctx = api.Context(0)
    d = fields.DeviceProblem(p, torch.float64)
    vx0, vy0 = I.random_velocity(p, 21, 1e-3)
    p0 = np.random.default_rng(nx).standard_normal((ny, nx))
    vx, vy = d.velocity(vx0, vy0)
    pt = d.field(p0)
    pt[ny:] = float("nan")  # outside the cells: neither read into the mean nor written
    pt[:, nx:] = float("nan")
    api.uzawa_pressure(ctx, d.grid, vx, vy, d.eta_c, 0.6, pt)
    torch.cuda.synchronize()
    assert normwise(d.get_cell(pt), U.pressure_update(p, vx0, vy0, p0, 0.6)) <= 1e-13
    assert torch.isnan(pt[ny:]).all() and torch.isnan(pt[:, nx:]).all()
    ctx.close()
