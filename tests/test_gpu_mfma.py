"""Matrix-core spreading and interpolation against the global-memory kernels
(method GM-sort) of the same plan: every width that takes them, ragged grids,
one point, a few, groups that fill several chunks, several subproblems a bin."""
import numpy as np
import pytest
import torch

import workloads
from paper_2102_08463_amd import Plan

pytestmark = pytest.mark.gpu

# eps -> w = 8 .. 14, modes, points, kind
CASES = [(1e-7, (20, 24, 18), 5000, "uniform"), (1e-8, (13, 11, 9), 1, "uniform"),
         (1e-9, (40, 10, 33), 30000, "uniform"), (1e-10, (16, 16, 16), 3, "uniform"),
         (1e-11, (25, 30, 16), 17, "gaussian"), (1e-12, (41, 41, 41), 60000, "gaussian"),
         (1e-12, (20, 50, 12), 20000, "cluster"), (1e-13, (18, 17, 16), 9000, "uniform")]


@pytest.mark.parametrize("eps,modes,M,kind", CASES)
def test_f64_3d(eps, modes, M, kind):
    pts = [torch.from_numpy(a).cuda() for a in workloads.points(kind, M, 3, 11)]
    c = torch.from_numpy(workloads.strengths(M, 12)).cuda()
    out = {}
    for method in ("sm", "gmsort"):
        with Plan(1, modes, eps=eps, dtype=torch.complex128, method=method) as p:
            p.setpts(*pts)
            grid = p.spread(c)
            again = p.spread(c)
            field = torch.from_numpy(workloads.strengths(p.fine_shape, 13)).cuda()
            out[method] = (grid, p.interp(field))
            if method == "sm":
                assert torch.equal(torch.view_as_real(grid), torch.view_as_real(again))
                perm, _ = p.get_sort()
                f = p.execute(c)
                fs = p.execute_sorted(c[perm.long()].contiguous())
                assert torch.equal(torch.view_as_real(f), torch.view_as_real(fs))
    # both round each of the w^3 products and their sums: a few hundred roundings at most
    for a, b in zip(out["sm"], out["gmsort"]):
        err = torch.linalg.vector_norm(a - b) / torch.linalg.vector_norm(b)
        assert err <= 300 * 2.0 ** -53, float(err)
