"""The walk of a coarse level's two post-smoothing sweeps, where its regions are 16 and 32 per
CU (FP64, FP32): just above and below both lines, against the cycle run stage by stage, bit
for bit as in test_gpu_mg_passes.py, in levels narrower than a strip and of several.
"""
import pytest
import torch

from test_gpu_mg_passes import ctx, problem, vcycle  # noqa: F401 (ctx: fixture)

pytestmark = pytest.mark.gpu


# level 1 has 16.7 and 15.6, 32.7 and 31.99, 16.1 and 32.3 regions of 12 x 12 per CU of 256
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nx,ny", [(1640, 1480), (1640, 1384), (2184, 2176), (2152, 2160), (40, 49600),
                                   (40, 99200)])
def test_walk_up_equals_the_stages(ctx, nx, ny, dtype):  # noqa: F811
    p = problem(nx, ny)
    got = vcycle(ctx, p, dtype, 1, max_levels=3)
    ref = vcycle(ctx, p, dtype, 1, max_levels=3, coarse_smoother="ras", coarse_tile=8, coarse_k=2, coarse_halo=2)
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
