"""The quotients of the energy norms, r^2 / d and f^2 / d, are rounded once: on problems
whose diagonals are exact (whole viscosities, cells of powers of two) and whose force has a
single entry, at rest, N_v = N_f is that one quotient, equal to the oracle's division bit
for bit.  Entries far from 1 and viscosities far from 1 among them: their squares and
quotients stay in the format's range down to its subnormal numbers.
"""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from oracle import stokes as S
from oracle import stokes3d as S3
from paper_2509_19061_amd import inputs as I

pytestmark = pytest.mark.gpu

# (exponent of the viscosities, of the force), base 2
SCALES = {torch.float64: [(0, 0), (-300, -300), (300, 400), (0, 505), (0, -520), (-600, 120), (900, 500)],
          torch.float32: [(0, 0), (-30, -60), (30, 50)]}


@pytest.fixture(scope="module")
def ctx():
    from paper_2509_19061_amd import api
    c = api.Context(0)
    yield c
    c.close()


def whole(rng, shape, scale):
    return rng.integers(1, 1 << 12, shape).astype(np.float64) * 2.0 ** scale


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("dx,dy", [(0.25, 0.25), (0.5, 0.125)])
def test_one_entry_2d(ctx, dx, dy, dtype):
    from paper_2509_19061_amd import api, fields
    rng = np.random.default_rng(7)
    nx, ny = 5, 4
    for es, fs in SCALES[dtype]:
        d = fields.DeviceProblem(SimpleNamespace(nx=nx, ny=ny, dx=dx, dy=dy, eta_c=whole(rng, (ny, nx), es),
                                                 eta_n=whole(rng, (ny + 1, nx + 1), es), fx=np.zeros((ny, nx + 1)),
                                                 fy=np.zeros((ny + 1, nx))), dtype)
        p, (vx, vy) = d.prob, d.velocity()
        for n in range(40):
            fx, fy = np.zeros_like(p.fx), np.zeros_like(p.fy)
            value = np.ldexp(rng.uniform(1.0, 2.0), fs)
            value = float(torch.tensor(value, dtype=dtype))
            if n % 2:
                fx[rng.integers(0, ny), rng.integers(1, nx)] = value
            else:
                fy[rng.integers(1, ny), rng.integers(0, nx)] = -value
            e = api.energy_norm(ctx, dtype, d.grid, vx, vy, None, d.eta_c, d.eta_n, d.field(fx), d.field(fy),
                                allow_nonfinite=True)
            o = S.energy(p, np.zeros_like(fx), np.zeros_like(fy), fx, fy)
            assert e[2] == o[2] and e[0] == o[0], (es, fs, n, e, o)


@pytest.mark.parametrize("nx,ny,length", [(2, 2, 1.0), (63, 40, 1.0), (300, 517, 1.0), (130, 60, 2.0 ** -37),
                                          (61, 65, 2.0 ** 25)])
@pytest.mark.parametrize("contrast", [1.0, 1e6])
def test_fp32_fields_have_the_norms_of_the_same_fields_in_fp64(ctx, nx, ny, length, contrast):
    """Sums and quotients are FP64 for both, in one order, so N_v, N_p and N_f are the same bits
    on cells of any size, and where a field is 0, infinite or not a number."""
    from paper_2509_19061_amd import api, fields
    rng = np.random.default_rng(nx + ny)

    def f32(a):
        return np.asarray(a, np.float32).astype(np.float64)

    eta_c = f32(np.exp(rng.uniform(0, np.log(contrast) + 1e-9, (ny, nx))))
    eta_n = f32(np.exp(rng.uniform(0, np.log(contrast) + 1e-9, (ny + 1, nx + 1))))
    p = SimpleNamespace(nx=nx, ny=ny, dx=length / nx, dy=length / ny, eta_c=eta_c, eta_n=eta_n,
                        fx=f32(rng.standard_normal((ny, nx + 1))), fy=f32(rng.standard_normal((ny + 1, nx))))
    vx, vy = f32(rng.standard_normal((ny, nx + 1))), f32(rng.standard_normal((ny + 1, nx)))
    pr = f32(rng.standard_normal((ny, nx)))
    for case in ("plain", "zeros", "inf force", "nan velocity", "zero viscosity", "inf viscosity"):
        q = SimpleNamespace(**vars(p))
        x = vx.copy()
        q.fx, q.eta_c, q.eta_n = p.fx.copy(), p.eta_c.copy(), p.eta_n.copy()
        if case == "zeros":
            x[:], q.fx[:] = 0.0, 0.0
        elif case == "inf force":
            q.fx[ny // 2, 1] = np.inf
        elif case == "nan velocity":
            x[ny // 2, 1] = np.nan
        elif case == "zero viscosity":
            q.eta_c[:], q.eta_n[:] = 0.0, 0.0
        elif case == "inf viscosity":
            q.eta_c[0, 0] = np.inf
        out = []
        for dtype in (torch.float32, torch.float64):
            d = fields.DeviceProblem(q, dtype)
            out.append(api.energy_norm(ctx, dtype, d.grid, *d.velocity(x, vy), d.field(pr), d.eta_c, d.eta_n, d.fx,
                                       d.fy, allow_nonfinite=True))
        np.testing.assert_array_equal(out[0], out[1], err_msg=case)


# the second grid is large enough for the plane walk
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nx,ny,nz", [(4, 5, 3), (3, 2, 769)])
def test_one_entry_3d(ctx, nx, ny, nz, dtype):
    from paper_2509_19061_amd import api, fields
    rng = np.random.default_rng(8)
    for es, fs in SCALES[dtype]:
        p = I.Problem3(nx, ny, nz, 0.25, 0.5, 0.125, whole(rng, (nz, ny, nx), es),
                       whole(rng, (nz, ny + 1, nx + 1), es), whole(rng, (nz + 1, ny, nx + 1), es),
                       whole(rng, (nz + 1, ny + 1, nx), es), np.zeros((nz, ny, nx + 1)), np.zeros((nz, ny + 1, nx)),
                       np.zeros((nz + 1, ny, nx)))
        d = fields.DeviceProblem3(p, dtype)
        v = d.velocity()
        for n in range(40):
            f = [np.zeros_like(p.fx), np.zeros_like(p.fy), np.zeros_like(p.fz)]
            at = [rng.integers(0, nz), rng.integers(0, ny), rng.integers(0, nx)]
            at[2 - n % 3] = rng.integers(1, (nx, ny, nz)[n % 3])  # not on the component's walls
            f[n % 3][tuple(at)] = float(torch.tensor(np.ldexp(rng.uniform(1.0, 2.0), fs), dtype=dtype))
            e = api.energy_norm3d(ctx, dtype, d.grid, v, d.eta, d.velocity(f))
            o = S3.energy(p, *(np.zeros_like(a) for a in f), *f)
            assert e[1] == o[1] and e[0] == o[0], (es, fs, n, e, o)
