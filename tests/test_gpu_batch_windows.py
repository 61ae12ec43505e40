"""Windows of a batch's points: a point next to the edge of a kernel window takes
the taps that its transform's own plan takes, whatever bins the batch shares."""
import math

import numpy as np
import pytest

from tests.gpu_helpers import note

pytestmark = pytest.mark.gpu

N = 250                      # 500^2 cells: own bins 16 x 16, shared by four or more 32 x 32
CELLS = 2 * N


def _edge_points(w, count):
    """Coordinates within a few single precision units of the edge of a window
    (half a cell for odd w, a whole one for even), next to x = 0, where
    single precision coordinates are fine enough; the cell lies in the upper
    half of a 32-cell bin."""
    j = np.arange(count)
    off = (0.5 if w % 2 else 1.0) + (j - count // 2) * (4e-6 / count)
    gx = CELLS // 2 + off
    gy = CELLS // 2 + 1.0 + off[::-1]
    return [((g / CELLS) * 2 * math.pi - math.pi).astype(np.float32) for g in (gx, gy)]


# Batch and plan differ by the rounding of their FFTs: 18 butterfly levels of
# 2^-24, up to ten times that at the band's corner, 1.1e-5.  A window that is off
# by one cell moves a value by exp(-2.3 w): 1e-2, 1e-3 and 1e-4.
TOL = 3e-5


@pytest.mark.parametrize("eps,w", [(1e-1, 2), (1e-2, 3), (1e-3, 4)])
def test_type2_points_at_window_edges(eps, w):
    import torch
    from paper_2102_08463_amd import Batch, Plan
    note(f"batch windows type 2 w={w}")
    T, M = 4, 4000
    x = [torch.from_numpy(a).cuda() for a in _edge_points(w, M)]
    f = torch.view_as_complex(torch.randn(T, N, N, 2, generator=torch.Generator().manual_seed(3))).cuda()
    with Batch(2, [(N, N)] * T, [M] * T, eps=eps) as b:
        b.setpts(*[v.repeat(T) for v in x])
        got = b.execute(f.reshape(-1)).reshape(T, M)
    for t in range(T):
        with Plan(2, (N, N), eps=eps) as p:
            assert p.info()["w"] == w and p.info()["binsize"][:2] == [16, 16]
            want = p.setpts(*x).execute(f[t].contiguous())
        rms = float(torch.linalg.norm(want)) / math.sqrt(M)
        assert float((got[t] - want).abs().max()) <= TOL * max(rms, float(f[t].abs().mean())), t


@pytest.mark.parametrize("eps,w", [(1e-2, 3), (1e-3, 4)])
def test_type1_points_at_window_edges(eps, w):
    import torch
    from paper_2102_08463_amd import Batch, Plan
    note(f"batch windows type 1 w={w}")
    T = 40                   # one point each, so that every mode has modulus one
    x = [torch.from_numpy(a).cuda() for a in _edge_points(w, T)]
    c = torch.ones(T, dtype=torch.complex64, device="cuda")
    with Batch(1, [(N, N)] * T, [1] * T, eps=eps) as b:
        b.setpts(*x)
        got = b.execute(c).reshape(T, N, N)
    for t in range(T):
        with Plan(1, (N, N), eps=eps) as p:
            want = p.setpts(*[v[t:t + 1].contiguous() for v in x]).execute(c[:1].contiguous())
        assert float((got[t] - want).abs().max()) <= TOL, t


def test_given_extent_keeps_the_others():
    """A transform with one extent given keeps its plan's other one: next to a
    512-cell side the batch's 32 cells would not fit in LDS."""
    import torch
    from paper_2102_08463_amd import Batch, Plan
    note("batch, one extent given")
    T, M, n = 4, 2000, 256
    g = torch.Generator().manual_seed(5)
    x = [((torch.rand(T * M, generator=g) * 2 - 1) * math.pi).cuda() for _ in range(2)]
    c = torch.view_as_complex(torch.randn(T * M, 2, generator=g)).cuda()
    with Batch(1, [(n, n)] * T, [M] * T, eps=1e-5, binsize=[(512, 0)] + [(0, 0)] * (T - 1)) as b:
        b.setpts(*x)
        got = b.execute(c).reshape(T, -1)
    for t in range(T):
        with Plan(1, (n, n), eps=1e-5) as p:
            sl = slice(t * M, t * M + M)
            want = p.setpts(*[v[sl].contiguous() for v in x]).execute(c[sl].contiguous()).reshape(-1)
        assert float(torch.linalg.norm(got[t] - want) / torch.linalg.norm(want)) <= 2e-4, t
