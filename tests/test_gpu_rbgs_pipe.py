"""Pipelined red-black Gauss-Seidel (K sweeps in registers per pass over memory)
against the CPU oracle, at the edges of the strips (63 - 6 K columns), of the row
segments and of the grid, on square and other cells, with and without a pressure.

Bars: FP64 normwise 1e-12; FP32 1e-5 per sweep from the same state rounded to FP32.
The passes are exact in number: any split of the sweeps gives the same bits, and so do
the in-place half-sweeps that a captured stream without scratch takes.
"""
import pytest
import torch

from gpu_util import as_dtype, normwise
from oracle import stokes as S
from paper_2509_19061_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2509_19061_amd import api
    c = api.Context(0)
    yield c
    c.close()


def problem(nx, ny, dtype):
    p = I.sinker_problem(nx, ny, [(0.3, 0.4, 0.2), (0.7, 0.6, 0.15)], 1e4, 1.0)
    for f in ("eta_c", "eta_n", "fx", "fy"):
        setattr(p, f, as_dtype(getattr(p, f), dtype))
    vx, vy = I.random_velocity(p, nx + ny, 1e-2)
    return p, as_dtype(vx, dtype), as_dtype(vy, dtype)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nx,ny", [(2, 2), (3, 41), (50, 5), (51, 51), (57, 7), (58, 58), (200, 130), (701, 12),
                                   (12, 701)])
def test_sweeps_match_oracle(ctx, nx, ny, dtype):
    from paper_2509_19061_amd import api, fields
    p, vx0, vy0 = problem(nx, ny, dtype)
    dp = fields.DeviceProblem(p, dtype)
    ox, oy = vx0, vy0
    bx, by = S.rhs(p, p.fx, p.fy)
    for sweeps in range(1, 6):
        ox, oy = S.rbgs(p, bx, by, 1.0, ox, oy)
        vx, vy = dp.velocity(vx0, vy0)
        api.smooth(ctx, dtype, dp.grid, vx, vy, None, dp.eta_c, dp.eta_n, dp.fx, dp.fy, sweeps, "rbgs")
        tol = 1e-12 if dtype == torch.float64 else sweeps * 1e-5
        assert normwise(dp.get_vx(vx), ox) <= tol and normwise(dp.get_vy(vy), oy) <= tol, sweeps


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nx,ny", [(300, 200), (257, 257)])
def test_any_split_and_the_half_sweeps_give_the_same_bits(nx, ny, dtype):
    from paper_2509_19061_amd import api, fields
    p, vx0, vy0 = problem(nx, ny, dtype)
    dp = fields.DeviceProblem(p, dtype)
    out = []
    for sweeps, calls in ((7, 1), (1, 7)):
        c = api.Context(0)
        vx, vy = dp.velocity(vx0, vy0)
        for _ in range(calls):
            api.smooth(c, dtype, dp.grid, vx, vy, None, dp.eta_c, dp.eta_n, dp.fx, dp.fy, sweeps, "rbgs", omega=1.2)
        torch.cuda.synchronize()
        assert c.scratch_bytes() > 0
        out.append((vx, vy))
        c.close()
    vx, vy = dp.velocity(vx0, vy0)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    c = api.Context(0)
    c.set_stream(s)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):  # a first call: the context has no scratch and may get none
        api.smooth(c, dtype, dp.grid, vx, vy, None, dp.eta_c, dp.eta_n, dp.fx, dp.fy, 7, "rbgs", omega=1.2)
    assert c.scratch_bytes() == 0
    g.replay()
    torch.cuda.synchronize()
    for v in (out[1], (vx, vy)):
        assert torch.equal(out[0][0], v[0]) and torch.equal(out[0][1], v[1])
    c.close()
