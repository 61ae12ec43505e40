"""Stacked transforms (n_trans > 1) share their launches: each must equal the
same transform run alone, bit for bit, also when the tile scratch holds only
some of them (3D, 128^3 grid: three at a time)."""
import pytest
import torch

import workloads
from paper_2102_08463_amd import Plan

pytestmark = pytest.mark.gpu

CASES = [((40, 33), 3, torch.complex64, 1e-5), ((64, 64, 64), 5, torch.complex64, 1e-4),
         ((30, 20, 25), 3, torch.complex128, 1e-9), ((500,), 4, torch.complex64, 1e-5),
         ((20, 31), 2, torch.complex128, 1e-8), ((6, 7, 5), 3, torch.complex128, 1e-4)]


@pytest.mark.parametrize("modes,T,dtype,eps", CASES)
def test_each_equals_alone(modes, T, dtype, eps):
    dim, M = len(modes), 20000
    rt = torch.float32 if dtype == torch.complex64 else torch.float64
    pts = [torch.from_numpy(a).to(rt).cuda() for a in workloads.gaussian(M, dim, 1, 0.6)]
    c = torch.from_numpy(workloads.strengths((T, M), 2)).to(dtype).cuda()
    f = torch.from_numpy(workloads.strengths((T,) + modes[::-1], 3)).to(dtype).cuda()
    with Plan(1, modes, T, eps, dtype=dtype) as p, Plan(1, modes, 1, eps, dtype=dtype) as one:
        p.setpts(*pts)
        one.setpts(*pts)
        for _ in range(2):
            got, back = p.execute(c), p.execute_adjoint(f)
            for t in range(T):
                assert torch.equal(torch.view_as_real(got[t]),
                                   torch.view_as_real(one.execute(c[t].contiguous())))
                assert torch.equal(torch.view_as_real(back[t]),
                                   torch.view_as_real(one.execute_adjoint(f[t].contiguous())))
