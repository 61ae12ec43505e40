"""Interpolation reads its plan alone: graphs of two calls may be replayed on two
streams at once, and eager calls beside them."""
import math

import pytest

from tests.gpu_helpers import note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [1e-7, 1e-12])
def test_two_graphs_at_once(eps):
    import torch
    from paper_2102_08463_amd import Plan
    note(f"concurrent interp {eps}")
    M, modes = 200000, (40, 36, 44)
    g = torch.Generator(device="cuda").manual_seed(2)
    x = [(torch.rand(M, generator=g, device="cuda", dtype=torch.float64) * 2 - 1) * math.pi
         for _ in range(3)]
    with Plan(2, modes, eps=eps, dtype=torch.complex128) as p:
        p.setpts(*x)
        grids = [torch.view_as_complex(torch.randn(*p.fine_shape, 2, generator=g, device="cuda",
                                                   dtype=torch.float64)) for _ in range(3)]
        want = [p.interp(a).clone() for a in grids]
        torch.cuda.synchronize()
        s = torch.cuda.Stream()
        p.set_stream(s)
        graphs, outs = [], []
        for a in grids[:2]:
            gr = torch.cuda.CUDAGraph()
            with torch.cuda.graph(gr, stream=s):
                outs.append(p.interp(a))
            graphs.append(gr)
        side = [torch.cuda.Stream(), torch.cuda.Stream()]
        for _ in range(5):
            for k in range(2):
                with torch.cuda.stream(side[k]):
                    graphs[k].replay()
            with torch.cuda.stream(s):
                third = p.interp(grids[2])
            torch.cuda.synchronize()
            for got, ref in zip(outs + [third], want):
                assert torch.equal(torch.view_as_real(got), torch.view_as_real(ref))
        # the plan's own type 2 afterwards
        f = torch.view_as_complex(torch.randn(*modes[::-1], 2, generator=g, device="cuda",
                                              dtype=torch.float64))
        with torch.cuda.stream(s):
            again = p.execute(f)
        torch.cuda.synchronize()
        with Plan(2, modes, eps=eps, dtype=torch.complex128) as q:
            ref = q.setpts(*x).execute(f)
        assert torch.equal(torch.view_as_real(again), torch.view_as_real(ref))
