"""Red-black Gauss-Seidel captured on a context that already holds its scratch: the graph
works in place on the caller's arrays, so later and larger calls on the context, which
regrow the scratch, leave its replays alone; nor does it take the scratch from graphs of the
other smoothers.  Replays give the bits of the uncaptured call.
"""
import pytest
import torch

from paper_2509_19061_amd import inputs as I

pytestmark = pytest.mark.gpu


def problem(n, dtype):
    from paper_2509_19061_amd import fields
    p = I.sinker_problem(n, n - 7, [(0.3, 0.4, 0.2), (0.7, 0.6, 0.15)], 1e4, 1.0)
    return p, fields.DeviceProblem(p, dtype)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("variant,sweeps", [("rbgs", 2), ("rbgs", 7), ("jacobi_fused", 25)])
def test_replays_outlive_larger_calls(variant, sweeps, dtype):
    from paper_2509_19061_amd import api
    p, d = problem(130, dtype)
    big = problem(400, dtype)[1]
    v0 = I.random_velocity(p, 3, 1e-2)
    s = torch.cuda.Stream()
    c = api.Context(0)
    c.set_stream(s)
    torch.cuda.synchronize()

    def call(v):
        api.smooth(c, dtype, d.grid, *v, None, d.eta_c, d.eta_n, d.fx, d.fy, sweeps, variant)

    with torch.cuda.stream(s):
        ref, v = d.velocity(*v0), d.velocity(*v0)
        start = [t.clone() for t in v]
        call(ref)  # the context holds scratch from here on
        s.synchronize()
        held = c.scratch_bytes()
        assert held > 0
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            call(v)
        for _ in range(3):
            for a, b in zip(v, start):
                a.copy_(b)
            # a larger Gauss-Seidel call: its scratch grows, and only its own
            w = big.velocity()
            api.smooth(c, dtype, big.grid, *w, None, big.eta_c, big.eta_n, big.fx, big.fy, 9, "rbgs")
            s.synchronize()
            filler = [torch.full((1 << 18,), 3.0, device="cuda") for _ in range(8)]
            g.replay()
            s.synchronize()
            assert torch.equal(v[0], ref[0]) and torch.equal(v[1], ref[1])
            assert all(bool((f == 3.0).all()) for f in filler)
    assert c.scratch_bytes() > held
    c.close()
