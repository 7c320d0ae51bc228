"""Calls whose velocity and right-hand side are the same memory: the right-hand side is what
the arrays hold when the call is made, so the result is bit for bit that of separate arrays.
"""
import pytest
import torch

from paper_2509_19061_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2509_19061_amd import api
    c = api.Context(0)
    yield c
    c.close()


def problem(nx, ny, dtype):
    from paper_2509_19061_amd import fields
    p = I.sinker_problem(nx, ny, [(0.3, 0.4, 0.2), (0.7, 0.6, 0.15)], 1e4, 1.0)
    d = fields.DeviceProblem(p, dtype)
    return p, d, d.velocity(*I.random_velocity(p, nx + ny, 1e-2))


# which arrays of (vx, vy) the right-hand side's (x, y) are; None: one of its own
SHARED = [(0, 1), (0, None), (None, 1), (1, 0)]


# strips of the finest level are 54 to 58 columns, its segments some rows: one and several
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nx,ny", [(16, 16), (132, 96), (512, 384)])
@pytest.mark.parametrize("shared", SHARED)
def test_vcycle(ctx, nx, ny, dtype, shared):
    from paper_2509_19061_amd import api, fields
    p, d, v0 = problem(nx, ny, dtype)
    d64 = fields.DeviceProblem(p, torch.float64)
    m = api.MG(ctx, d64.grid, d64.eta_c, d64.eta_n)
    out = []
    for apart in (True, False):
        v = [t.clone() for t in v0]
        b = [f if s is None else v[s].clone() if apart else v[s] for s, f in zip(shared, (d.fx, d.fy))]
        m.vcycle(dtype, *v, *b)
        out.append(v)
    torch.cuda.synchronize()
    m.close()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


# one to three passes of the pipelined sweeps; thin overlap and tiles of one pass each
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nx,ny", [(33, 20), (700, 500)])
@pytest.mark.parametrize("variant,opts", [("jacobi", {}), ("jacobi_fused", {}), ("ras", {}),
                                          ("ras", dict(k=4, halo=0, tile_x=32, tile_y=32))])
@pytest.mark.parametrize("sweeps", [1, 4, 9, 21])
def test_smooth(ctx, nx, ny, dtype, variant, opts, sweeps):
    from paper_2509_19061_amd import api
    p, d, v0 = problem(nx, ny, dtype)
    for shared in SHARED:
        out = []
        for apart in (True, False):
            v = [t.clone() for t in v0]
            b = [f if s is None else v[s].clone() if apart else v[s] for s, f in zip(shared, (d.fx, d.fy))]
            api.smooth(ctx, dtype, d.grid, *v, None, d.eta_c, d.eta_n, *b, sweeps, variant, **opts)
            out.append(v)
        torch.cuda.synchronize()
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1]), shared


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nx,ny", [(33, 20), (300, 200)])
def test_red_black_takes_the_running_values(ctx, nx, ny, dtype):
    """f = v: the value of an unknown when it is relaxed, colour by colour."""
    from gpu_util import normwise
    from oracle import stokes as S
    from paper_2509_19061_amd import api
    p, d, v = problem(nx, ny, dtype)
    ox, oy = d.get_vx(v[0]), d.get_vy(v[1])
    (cx, cy), sweeps = d.velocity(ox, oy), 4
    api.smooth(ctx, dtype, d.grid, cx, cy, None, d.eta_c, d.eta_n, d.fx, d.fy, sweeps, "rbgs")  # warms the scratch
    api.smooth(ctx, dtype, d.grid, *v, None, d.eta_c, d.eta_n, *v, sweeps, "rbgs", omega=0.9)
    torch.cuda.synchronize()
    # an unknown is relaxed once a sweep and read by others, never by itself, so its value at
    # that time is the one that the sweep starts from
    for _ in range(sweeps):
        ox, oy = S.rbgs(p, ox, oy, 0.9, ox, oy)
    tol = 1e-12 if dtype == torch.float64 else sweeps * 1e-5
    assert normwise(d.get_vx(v[0]), ox) <= tol and normwise(d.get_vy(v[1]), oy) <= tol
