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
