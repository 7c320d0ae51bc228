"""3D RAS with full overlap on small grids, where tiles in LDS take less time than the plane
walk: bit for bit the same number of Jacobi sweeps, on both sides of the line, for counts
that end in a partial iteration, with given shifts and the seed's.
"""
import numpy as np
import pytest
import torch

from paper_2509_19061_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("dims", [(2, 2, 2), (4, 4, 4), (9, 5, 7), (16, 16, 16), (33, 20, 4), (40, 40, 40)])
@pytest.mark.parametrize("tile,k,halo", [(8, 2, -1), (4, 3, 2), (3, 1, 0), (4, 2, 2), (2, 4, 3)])
def test_full_overlap_is_jacobi(dims, tile, k, halo, dtype):
    from paper_2509_19061_amd import api, fields
    ctx = api.Context(0)
    p = I.sinker_problem3d(*dims, [(0.4, 0.6, 0.5, 0.25)], 1e3, 1.0)
    d = fields.DeviceProblem3(p, dtype)
    v0 = I.random_velocity3d(p, 3, 1e-3)
    for sweeps in (1, 2, 7):
        ref, got, cut = d.velocity(v0), d.velocity(v0), d.velocity(v0)
        api.smooth3d(ctx, dtype, d.grid, ref, d.eta, d.f, sweeps, "jacobi_fused")
        api.smooth3d(ctx, dtype, d.grid, got, d.eta, d.f, sweeps, "ras", tile=tile, k=k, halo=halo, seed=5)
        shifts = np.arange(3 * sweeps, dtype=np.int32).reshape(-1, 3)
        api.smooth3d(ctx, dtype, d.grid, cut, d.eta, d.f, sweeps, "ras", tile=tile, k=k, halo=halo, shifts=shifts)
        torch.cuda.synchronize()
        for a, b, c in zip(d.get_v(ref), d.get_v(got), d.get_v(cut)):
            assert np.array_equal(a, b) and np.array_equal(a, c), sweeps
    ctx.close()


@pytest.mark.parametrize("dims", [(4, 4, 4), (40, 40, 40)])
@pytest.mark.parametrize("halo", [-1, 1, 0])
def test_negative_shifts_are_refused(dims, halo):
    """Wherever the iterations run, and before anything is written; multiples of the tile are 0."""
    from paper_2509_19061_amd import api, fields
    ctx = api.Context(0)
    p = I.sinker_problem3d(*dims, [(0.4, 0.6, 0.5, 0.25)], 1e3, 1.0)
    d = fields.DeviceProblem3(p, torch.float64)
    v0 = I.random_velocity3d(p, 3, 1e-3)
    v, before = d.velocity(v0), d.velocity(v0)
    for bad in ([[-1, 0, 0], [0, 0, 0]], [[0, 0, 0], [0, 3, -5]]):
        with pytest.raises(api.StkError) as e:
            api.smooth3d(ctx, torch.float64, d.grid, v, d.eta, d.f, 4, "ras", tile=4, k=2, halo=halo,
                         shifts=np.array(bad))
        assert e.value.code == api.EINVAL
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(v, before))
    api.smooth3d(ctx, torch.float64, d.grid, v, d.eta, d.f, 4, "ras", tile=4, k=2, halo=halo,
                 shifts=np.array([[-4, 0, 0], [0, 3, -8]]))
    torch.cuda.synchronize()
    ctx.close()
