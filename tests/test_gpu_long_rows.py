"""Rows too long for the 32-bit windows of the pipelined passes (192 of them are 4 GiB: a
row stride of 23 MB), on small grids: the kernels that gather or stage their operands take
over, and the results are those of the same problem in short rows.

Bit for bit where those kernels compute the same expressions (Jacobi, Gauss-Seidel, RAS
with full overlap, V-cycles); thin overlaps normwise 1e-13 and 1e-6, a rounding per sweep.
"""
import pytest
import torch

from gpu_util import normwise
from paper_2509_19061_amd import inputs as I

pytestmark = pytest.mark.gpu

ROW = 23 << 20  # bytes
SINKERS = [(0.3, 0.4, 0.2), (0.7, 0.6, 0.15)]


@pytest.fixture(scope="module")
def ctx():
    from paper_2509_19061_amd import api
    c = api.Context(0)
    yield c
    c.close()


def long(t, ld):
    out = torch.zeros((t.shape[0], ld), dtype=t.dtype, device=t.device)
    out[:, :t.shape[1]] = t
    return out


def short(t, like):
    return t[:, :like.shape[1]].contiguous()


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nx,ny", [(2, 2), (70, 3), (33, 20)])
def test_smoothers(ctx, nx, ny, dtype):
    from paper_2509_19061_amd import api, fields
    from paper_2509_19061_amd._lib import Grid
    p = I.sinker_problem(nx, ny, SINKERS, 1e3, 1.0)
    d = fields.DeviceProblem(p, dtype)
    v0, pr = I.random_velocity(p, 1, 1e-2), d.field(I.random_pressure(p, 2))
    ld = ROW // pr.element_size()
    grid = Grid(nx, ny, ld, float(p.dx), float(p.dy))
    far = [long(t, ld) for t in (pr, d.eta_c, d.eta_n, d.fx, d.fy)]
    for variant, opts in (("jacobi", {}), ("jacobi_fused", {}), ("rbgs", {}), ("ras", dict(k=3, tile_x=16, tile_y=16)),
                          ("ras", dict(k=4, halo=1, tile_x=16, tile_y=16))):
        for sweeps in (1, 6):
            a = d.velocity(*v0)
            b = [long(t, ld) for t in d.velocity(*v0)]
            api.smooth(ctx, dtype, d.grid, *a, pr, d.eta_c, d.eta_n, d.fx, d.fy, sweeps, variant, seed=3, **opts)
            api.smooth(ctx, dtype, grid, *b, *far, sweeps, variant, seed=3, **opts)
            torch.cuda.synchronize()
            for x, y in zip(a, b):
                y = short(y, x)
                if "halo" in opts:
                    assert normwise(y.double().cpu().numpy(), x.double().cpu().numpy()) <= \
                        (1e-13 if dtype == torch.float64 else 1e-6), (variant, sweeps)
                else:
                    assert torch.equal(x, y), (variant, sweeps)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nu", [1, 2, 3])
def test_vcycle(ctx, nu, dtype):
    from paper_2509_19061_amd import api, fields
    from paper_2509_19061_amd._lib import Grid
    nx, ny = 16, 8
    p = I.sinker_problem(nx, ny, SINKERS, 1e3, 1.0)
    d64, d = fields.DeviceProblem(p, torch.float64), fields.DeviceProblem(p, dtype)
    ld = ROW // d.fx.element_size()
    m = api.MG(ctx, d64.grid, d64.eta_c, d64.eta_n, nu1=nu, nu2=nu, coarsest=4)
    far = api.MG(ctx, Grid(nx, ny, ld, float(p.dx), float(p.dy)), long(d64.eta_c, ld), long(d64.eta_n, ld), nu1=nu,
                 nu2=nu, coarsest=4)
    a, b = d.velocity(*I.random_velocity(p, 1, 1e-2)), (d.fx, d.fy)
    fa, fb = [long(t, ld) for t in a], [long(t, ld) for t in b]
    for _ in range(2):
        m.vcycle(dtype, *a, *b)
        far.vcycle(dtype, *fa, *fb)
    torch.cuda.synchronize()
    for x, y in zip(a, fa):
        assert torch.equal(x, short(y, x))
    m.close()
    far.close()
