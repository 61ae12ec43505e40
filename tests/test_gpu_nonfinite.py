"""Infinities and NaN in double precision 3D spreading and interpolation stay where
the kernel's support carries them, on the matrix cores as tap by tap."""
import math

import numpy as np
import pytest

from tests.gpu_helpers import note

pytestmark = pytest.mark.gpu

# sums of up to a few thousand terms in two orders, relative to the largest
TOL = 4000 * 2.0 ** -53


def _plan(eps, M, seed=4):
    import torch
    from paper_2102_08463_amd import Plan
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = [(torch.rand(M, generator=g, device="cuda", dtype=torch.float64) * 2 - 1) * math.pi
         for _ in range(3)]
    p = Plan(1, (24, 20, 28), eps=eps, dtype=torch.complex128)
    p.setpts(*x)
    return p, x, g


def _near(p, x, cell, other):
    """Whether the support of points at x covers grid cell ``cell`` (integers):
    w cells from the first at or above x - w / 2, wrapped."""
    inf = p.info()
    w, n = inf["w"], inf["nfine"][:3]
    ok = np.ones(other, dtype=bool)
    for d in range(3):
        g = (x[d].cpu().numpy() + math.pi) * n[d] / (2 * math.pi)
        ok &= (cell[d] - np.ceil(g - w / 2)) % n[d] < w
    return ok


@pytest.mark.parametrize("eps", [1e-7, 1e-9, 1e-12])
@pytest.mark.parametrize("bad", [complex(math.nan, 0), complex(0, math.inf), complex(-math.inf, math.nan)])
def test_spread_keeps_to_the_support(eps, bad):
    import torch
    M = 3000
    note(f"nonfinite spread {eps} {bad}")
    p, x, g = _plan(eps, M)
    c = torch.view_as_complex(torch.randn(M, 2, generator=g, device="cuda", dtype=torch.float64))
    hit = [5, 6, 1700]
    zero = c.clone()
    zero[hit] = 0
    c[hit] = bad
    got, want = p.spread(c).cpu().numpy(), p.spread(zero).cpu().numpy()
    inf = p.info()
    w, n = inf["w"], inf["nfine"][:3]
    inside = np.zeros(got.shape, dtype=bool)
    for j in hit:
        idx = []
        for d in range(3):
            gd = (float(x[d][j]) + math.pi) * n[d] / (2 * math.pi)
            idx.append((int(math.ceil(gd - w / 2)) + np.arange(w)) % n[d])
        inside[np.ix_(idx[2], idx[1], idx[0])] = True
    assert not np.isfinite(got[inside]).any()
    assert np.isfinite(got[~inside]).all()
    assert np.abs(got - want)[~inside].max() <= TOL * np.abs(want).max()
    p.destroy()


@pytest.mark.parametrize("eps", [1e-7, 1e-9, 1e-12])
@pytest.mark.parametrize("bad", [complex(math.nan, 1), complex(1, math.inf)])
def test_interp_keeps_to_the_support(eps, bad):
    import torch
    M = 3000
    note(f"nonfinite interp {eps} {bad}")
    p, x, g = _plan(eps, M)
    grid = torch.view_as_complex(torch.randn(*p.fine_shape, 2, generator=g, device="cuda",
                                             dtype=torch.float64))
    cell = (17, 3, 40)
    zero = grid.clone()
    zero[cell[2], cell[1], cell[0]] = 0
    grid[cell[2], cell[1], cell[0]] = bad
    got, want = p.interp(grid).cpu().numpy(), p.interp(zero).cpu().numpy()
    near = _near(p, x, cell, M)
    assert 0 < near.sum() < M
    assert not np.isfinite(got[near]).any() and np.isfinite(got[~near]).all()
    assert np.abs(got - want)[~near].max() <= TOL * np.abs(want).max()
    # a finite grid again: the flag of one item does not stay for the next
    assert np.isfinite(p.interp(zero).cpu().numpy()).all()
    p.destroy()
