"""Residual and norms on grids whose waves walk 16 rows (4096 waves or more: strips of 62
columns times segments), ragged in both directions, against the CPU oracle; and the
right-hand side that the norm's pass stores there for the next V-cycle, against the pass
that forms it alone.  Smaller grids, whose waves walk 8 rows, are covered beside the kernels.

Bars: residual normwise 1e-12 (FP64), 1e-5 (FP32, formed in FP32); norms, whose sums are
FP64 for both, relative 1e-9 (8e6 positive terms, each sum within n eps).
"""
import numpy as np
import pytest
import torch

from gpu_util import as_dtype, normwise
from oracle import stokes as S
from paper_2509_19061_amd import inputs as I

pytestmark = pytest.mark.gpu

SINKERS = [(0.4, 0.6, 0.1), (0.65, 0.35, 0.08)]


def waves(nx, ny, rows):
    return -(-(nx + 1) // 62) * -(-(ny + 1) // rows)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("with_p", [False, True])
@pytest.mark.parametrize("nx,ny", [(2050, 2061), (61, 65551), (4033, 992)])
def test_sixteen_row_walks_match_oracle(nx, ny, with_p, dtype):
    from paper_2509_19061_amd import api, fields
    assert waves(nx, ny, 16) >= 4096
    ctx = api.Context(0)
    p = I.sinker_problem(nx, ny, SINKERS, 1e2, 1.0)
    for f in ("eta_c", "eta_n", "fx", "fy"):
        setattr(p, f, as_dtype(getattr(p, f), dtype))
    vx, vy = (as_dtype(v, dtype) for v in I.random_velocity(p, 3, 1e-2))
    pr = as_dtype(I.random_pressure(p, 4), dtype) if with_p else None
    d = fields.DeviceProblem(p, dtype)
    v, pt = d.velocity(vx, vy), d.field(pr) if with_p else None
    r, rp = d.velocity(), d.field()
    api.residual(ctx, dtype, d.grid, *v, pt, d.eta_c, d.eta_n, d.fx, d.fy, *r, rp)
    e = api.energy_norm(ctx, dtype, d.grid, *v, pt, d.eta_c, d.eta_n, d.fx, d.fy)
    ox, oy, op = S.residual(p, vx, vy, p.fx, p.fy, pr)
    tol = 1e-12 if dtype == torch.float64 else 1e-5
    for got, ref in ((d.get_vx(r[0]), ox), (d.get_vy(r[1]), oy), (d.get_cell(rp), op)):
        assert normwise(got, ref) <= tol
    np.testing.assert_allclose(e, S.energy(p, vx, vy, p.fx, p.fy, pr), rtol=1e-9)
    ctx.close()


@pytest.mark.parametrize("mode", ["f64", "f32_refined"])
@pytest.mark.parametrize("solver", ["uzawa", "anderson"])
def test_stored_right_hand_side_equals_a_pass_of_its_own(mode, solver):
    from paper_2509_19061_amd import api, fields
    nx, ny = 2060, 2068
    assert waves(nx, ny, 16) >= 4096
    p = I.sinker_problem(nx, ny, SINKERS, 1e2, 1.0)
    ctx = api.Context(0)
    d = fields.DeviceProblem(p, torch.float64)
    m = api.MG(ctx, d.grid, d.eta_c, d.eta_n, max_levels=2)  # (no small coarsest level to solve)
    run = api.uzawa_solve if solver == "uzawa" else lambda *a, **kw: api.uzawa_anderson(*a, depth=0, **kw)
    res = []
    for calls, cycles in ((1, 3), (3, 1)):
        vx, vy = d.velocity()
        pt = d.field()
        api.litho_pressure(ctx, d.grid, d.fy, pt)
        hist = []
        for _ in range(calls):
            hist += list(run(m, d.grid, vx, vy, pt, d.eta_c, d.eta_n, d.fx, d.fy, allow_notconv=True, tol=0.0,
                             max_cycles=cycles, mode=mode)[1][1:])
        torch.cuda.synchronize()
        res.append((vx, vy, pt, hist))
    assert res[0][3] == res[1][3]
    assert all(torch.equal(a, b) for a, b in zip(res[0][:3], res[1][:3]))
    m.close()
    ctx.close()
