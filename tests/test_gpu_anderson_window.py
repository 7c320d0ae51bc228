"""The Anderson window's memory stays with the context between calls up to a
size and belongs to the call beyond it: the steps' bits depend neither on what
an earlier call left in it nor on where it lies."""
import numpy as np
import pytest
import torch

from paper_2509_19061_amd import inputs as I

pytestmark = pytest.mark.gpu


def _steps(ctx, nx, ny, depth, mode, cycles):
    from paper_2509_19061_amd import api, fields
    p = I.sinker_problem(nx, ny, [(0.4, 0.6, 0.1), (0.65, 0.35, 0.08)], 1e2, 1.0)
    d = fields.DeviceProblem(p, torch.float64)
    m = api.MG(ctx, d.grid, d.eta_c, d.eta_n)
    vx, vy = d.velocity()
    pt = d.field()
    api.litho_pressure(ctx, d.grid, d.fy, pt)
    _, hist = api.uzawa_anderson(m, d.grid, vx, vy, pt, d.eta_c, d.eta_n, d.fx, d.fy, depth=depth, allow_notconv=True,
                                 tol=0.0, max_cycles=cycles, mode=mode)
    out = (d.get_vx(vx), d.get_vy(vy), d.get_cell(pt), np.asarray(hist))
    m.close()
    return out


# grows, shrinks, grows again; a window that turns over, one that does not fill, no steps
CALLS = [(64, 48, 2, "f64", 5), (132, 96, 3, "f32_refined", 6), (48, 64, 8, "f64", 3), (66, 40, 0, "f32_refined", 2),
         (64, 64, 3, "f64", 0), (192, 128, 4, "f64", 6)]


def test_kept_window_gives_the_bits_of_a_new_one():
    from paper_2509_19061_amd import api
    kept = api.Context(0)
    for call in CALLS:
        new = api.Context(0)
        for a, b in zip(_steps(kept, *call), _steps(new, *call)):
            assert np.array_equal(a, b), call
        new.close()
    kept.close()


def test_window_beyond_the_kept_size():
    """9 slots of 2048 x 2048 are 1.9 GB, 2 slots 0.4 GB: the same first steps, and only
    the small window stays."""
    from paper_2509_19061_amd import api
    hists, sizes = [], []
    for cycles in (2, 9):
        ctx = api.Context(0)
        hists.append(_steps(ctx, 2048, 2048, 8, "f64", cycles)[3])
        sizes.append(ctx.scratch_bytes())
        ctx.close()
    assert np.array_equal(hists[0], hists[1][:3])
    small = 2 * 6 * 2049 * 2049 * 8
    assert sizes[0] > small > sizes[1]
