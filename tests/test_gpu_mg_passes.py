"""The V-cycle's passes that hold several stages at once (the finest level's
sweeps with its residual, restriction and prolongation; both sweeps of a coarse
level's stage) against the same cycle run stage by stage: RAS with an overlap
that covers the sweeps' reach is the same smoother and takes the separate
kernels.  The values are bit for bit the same, so there is no tolerance.

Sizes: one tile or strip, an edge tile of one column or row (owned regions are
12 and 28 wide, strips 64 - 2 K), many strips and segments; 400 x 400 has more
than 256 small regions on its second level and takes the wide ones there; 1000 x 920
takes the walk down and regions up, 1640 x 1480 and 240 x 16384 the walk both ways (the
last with three strips, of which one has a single column).
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


def problem(nx, ny):
    return I.sinker_problem(nx, ny, [(0.3, 0.4, 0.2), (0.7, 0.6, 0.15)], 1e4, 1.0)


def vcycle(ctx, p, dtype, seed, **opts):
    from paper_2509_19061_amd import api, fields
    d64, d = fields.DeviceProblem(p, torch.float64), fields.DeviceProblem(p, dtype)
    m = api.MG(ctx, d64.grid, d64.eta_c, d64.eta_n, **opts)
    v, b = d.velocity(*I.random_velocity(p, seed, 1e-2)), d.velocity(*I.random_velocity(p, seed + 1, 1.0))
    for _ in range(2):  # the second cycle starts from the first one's velocity
        m.vcycle(dtype, *v, *b)
    torch.cuda.synchronize()
    m.close()
    return v


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nx,ny", [(20, 44), (44, 48), (56, 108), (64, 64), (120, 116), (236, 52), (400, 400),
                                   (1000, 920), (1640, 1480), (240, 16384)])
def test_two_sweeps_of_a_coarse_stage_in_one_pass(ctx, nx, ny, dtype):
    p = problem(nx, ny)
    cut = dict(max_levels=3) if nx * ny > 160000 else {}  # sizes that do not coarsen to a small grid
    got = vcycle(ctx, p, dtype, 1, **cut)
    ref = vcycle(ctx, p, dtype, 1, coarse_smoother="ras", coarse_tile=8, coarse_k=2, coarse_halo=2, **cut)
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nu1,nu2", [(1, 1), (2, 2), (3, 3), (1, 3), (3, 2)])
@pytest.mark.parametrize("nx,ny", [(20, 44), (56, 60), (64, 64), (236, 132)])
def test_finest_level_in_one_pass_each_way(ctx, nx, ny, nu1, nu2, dtype):
    p = problem(nx, ny)
    got = vcycle(ctx, p, dtype, 2, nu1=nu1, nu2=nu2)
    ref = vcycle(ctx, p, dtype, 2, nu1=nu1, nu2=nu2, fine_k=3, fine_halo=2)
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])


@pytest.mark.parametrize("mode", ["f64", "f32_refined"])
def test_batch_of_solves_equals_the_stage_by_stage_cycle(ctx, mode):
    from paper_2509_19061_amd import api, fields
    out = []
    for opts in ({}, dict(coarse_smoother="ras", coarse_tile=8, coarse_k=2, coarse_halo=2, fine_k=2, fine_halo=1)):
        ds = [fields.DeviceProblem(problem(*s), torch.float64) for s in ((64, 64), (96, 40), (20, 120))]
        ms = [api.MG(ctx, d.grid, d.eta_c, d.eta_n, **opts) for d in ds]
        vx, vy = [d.field() for d in ds], [d.field() for d in ds]
        rep = api.mg_solve_batch(ctx, ms, mode, vx, vy, None, [d.fx for d in ds], [d.fy for d in ds], tol=1e-6,
                                 max_iters=6, allow_notconv=True)
        out.append((vx + vy, [r["iterations"] for r in rep]))
        for m in ms:
            m.close()
    assert out[0][1] == out[1][1]
    assert all(torch.equal(a, b) for a, b in zip(out[0][0], out[1][0]))
