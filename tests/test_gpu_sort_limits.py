"""Bin-sort at the sizes where its kernels change: small blocks with summed
counts up to 262144 points, small blocks with scanned counts up to 2^20, large
blocks above; one bin, some, and more bins than the wave search takes."""
import numpy as np
import pytest

from oracle import binsort
from tests.gpu_helpers import make_points, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 63, 1023, 1024, 1025, 262144, 262145, 1 << 20, (1 << 20) + 1])
def test_permutation_bins_and_subproblems(M):
    from paper_2102_08463_amd import Plan
    note(f"sort limits {M}")
    pts64, pts = make_points("gaussian", M, 2, "f32", seed=5)
    for N, bs, method in (((20, 24), None, "auto"), ((600, 640), (6, 4), "gmsort"),
                          ((8, 8), (64, 64), "auto")):
        with Plan(1, N, eps=1e-4, binsize=bs, method=method) as p:
            p.setpts(*pts)
            inf = p.info()
            perm, start = p.get_sort()
            sub, _ = p.get_subproblems()
        keys = binsort.bin_keys(pts64, inf["nfine"][:2], inf["binsize"][:2])
        assert np.array_equal(perm.cpu().numpy(), binsort.permutation(keys))
        assert np.array_equal(start.cpu().numpy(), binsort.bin_starts(keys, inf["nbins"]))
        assert np.array_equal(sub[:, :3].cpu().numpy(),
                              binsort.subproblems(keys, inf["nbins"], inf["msub"]))


@pytest.mark.parametrize("M", [(1 << 20) + 1, 1 << 21, (1 << 21) + 5000])
def test_permutation_3d_wide_tiles(M):
    from paper_2102_08463_amd import Plan
    note(f"sort 3d {M}")
    pts64, pts = make_points("uniform", M, 3, "f32", seed=6)
    with Plan(1, (64, 60, 50), eps=1e-4) as p:
        p.setpts(*pts)
        inf = p.info()
        perm, start = p.get_sort()
    keys = binsort.bin_keys(pts64, inf["nfine"], inf["binsize"])
    assert np.array_equal(perm.cpu().numpy(), binsort.permutation(keys))
    assert np.array_equal(start.cpu().numpy(), binsort.bin_starts(keys, inf["nbins"]))


@pytest.mark.parametrize("M", [600, 300000, 2048 * 576 + 2047])
def test_kernels_cut_crowded_bins_finer(M):
    """The kernels cut bins finer than the list they report;
    all points in one bin, in more pieces than one merge group."""
    import torch
    import workloads
    from paper_2102_08463_amd import Plan
    note(f"crowded {M}")
    pts = [np.random.default_rng(7 + d).uniform(0.1, 0.2, M).astype(np.float32) for d in range(2)]
    c = workloads.strengths(M, seed=8).astype(np.complex64)
    eps = 1e-4
    with Plan(1, (24, 20), eps=eps, isign=-1, binsize=(32, 32)) as p:
        p.setpts(*[torch.from_numpy(a).cuda() for a in pts])
        inf = p.info()
        sub, _ = p.get_subproblems()
        f = p.execute(torch.from_numpy(c).cuda()).cpu().numpy()
    pts64 = [a.astype(np.float64) for a in pts]
    keys = binsort.bin_keys(pts64, inf["nfine"][:2], inf["binsize"][:2])
    assert np.array_equal(sub[:, :3].cpu().numpy(),
                          binsort.subproblems(keys, inf["nbins"], inf["msub"]))
    e1 = np.exp(-1j * np.outer(np.arange(24) - 12, pts64[0]))
    e2 = np.exp(-1j * np.outer(np.arange(20) - 10, pts64[1]))
    want = (e2 * c) @ e1.T
    # the requested accuracy, with the factor the kernel's error constant takes
    assert np.linalg.norm(f - want) <= 10 * eps * np.linalg.norm(want)


@pytest.mark.parametrize("M", [1, 255, 1536, 1537, 4096, 9000])
@pytest.mark.parametrize("sorted_order", [False, True])
def test_3d_bin_with_points_past_the_held_ones(M, sorted_order):
    """3D spreading keeps six points a thread (1536 a subproblem) and gathers
    the strengths of the rest again; all points in one bin, against the sums."""
    import torch
    import workloads
    from paper_2102_08463_amd import Plan
    note(f"held points {M} {sorted_order}")
    eps, N = 1e-5, (12, 10, 9)
    pts = [np.random.default_rng(9 + d).uniform(0.05, 0.2, M).astype(np.float32) for d in range(3)]
    c = workloads.strengths(M, seed=10).astype(np.complex64)
    with Plan(1, N, eps=eps, isign=-1, binsize=(16, 8, 8), msub=4096) as p:
        p.setpts(*[torch.from_numpy(a).cuda() for a in pts])
        ct = torch.from_numpy(c).cuda()
        if sorted_order:
            perm, _ = p.get_sort()
            f = p.execute_sorted(ct[perm.long()].contiguous())
        else:
            f = p.execute(ct)
        f = f.cpu().numpy()
    e = [np.exp(-1j * np.outer(np.arange(n) - n // 2, a.astype(np.float64)))
         for n, a in zip(N, pts)]
    want = np.einsum("zj,yj,xj->zyx", e[2], e[1], e[0] * c, optimize=True)
    assert np.linalg.norm(f - want) <= 10 * eps * np.linalg.norm(want)
