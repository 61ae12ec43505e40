"""A plan whose point set shrinks and grows again gives what a fresh plan gives:
the bin-sort and the subproblems take other shapes on either side of 2^20 points."""
import math

import pytest

from tests.gpu_helpers import note

pytestmark = pytest.mark.gpu

MI = 1 << 20


def _points(M, dim, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    return [(torch.rand(M, generator=g, device="cuda") * 2 - 1) * math.pi for _ in range(dim)]


@pytest.mark.parametrize("modes", [(96, 90), (24, 20, 28)])
@pytest.mark.parametrize("first", [MI + 1, 1_100_000])
def test_fewer_and_more_points(modes, first):
    import torch
    from paper_2102_08463_amd import Plan
    dim, eps = len(modes), 1e-5
    with Plan(1, modes, eps=eps) as p:
        for k, M in enumerate([first, MI, 1_000_000, 262_144, 1, first]):
            note(f"point counts {modes} {first} -> {M}")
            x = _points(M, dim, 10 + k)
            c = torch.view_as_complex(torch.randn(M, 2, device="cuda"))
            got = p.setpts(*x).execute(c)
            perm, start = p.get_sort()
            with Plan(1, modes, eps=eps) as q:
                want = q.setpts(*x).execute(c)
                qperm, qstart = q.get_sort()
            assert torch.equal(perm, qperm) and torch.equal(start, qstart)
            # (fixed-point tile sums: the same points give the same bits)
            assert torch.equal(torch.view_as_real(got), torch.view_as_real(want))


def test_fewer_points_type3():
    import torch
    from paper_2102_08463_amd import Plan
    with Plan(3, 2, eps=1e-5) as p:
        for k, (M, K) in enumerate([(MI + 1, MI + 1), (1_000_000, 900_000), (7, 1_000_000),
                                    (1_100_000, 5)]):
            note(f"point counts type 3 {M} {K}")
            x, s = _points(M, 2, 20 + k), [60 * a for a in _points(K, 2, 30 + k)]
            # (the corners keep the fine grid, and with it the plan's buffers)
            for a in x:
                a[0], a[-1] = -math.pi, math.pi
            for a in s:
                a[0], a[-1] = -180.0, 180.0
            c = torch.view_as_complex(torch.randn(M, 2, device="cuda"))
            got = p.setpts(*x, None, *s).execute(c)
            with Plan(3, 2, eps=1e-5) as q:
                want = q.setpts(*x, None, *s).execute(c)
            assert torch.equal(torch.view_as_real(got), torch.view_as_real(want))
