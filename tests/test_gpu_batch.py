"""Batched transforms of uneven sizes in one launch per stage, against the
exact sums and against one plan per transform."""
import numpy as np
import pytest

import workloads
from oracle import direct
from tests.gpu_helpers import note, rel_l2

pytestmark = pytest.mark.gpu


def _batch_inputs(n_modes, n_points, kinds, prec, seed):
    import torch
    rdt = np.float32 if prec == "f32" else np.float64
    cdt = np.complex64 if prec == "f32" else np.complex128
    pts = []
    for t, (M, kind) in enumerate(zip(n_points, kinds)):
        pts.append([np.asarray(a, dtype=rdt) for a in workloads.points(kind, M, len(n_modes[0]), seed + t)])
    cat = [np.concatenate([p[d] for p in pts]) if pts else np.zeros(0, rdt) for d in range(len(n_modes[0]))]
    tens = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in cat]
    return pts, tens, cdt


@pytest.mark.parametrize("prec,eps", [("f32", 1e-5), ("f64", 1e-11)])
@pytest.mark.parametrize("ntype", [1, 2])
def test_small_mixed_batch(prec, eps, ntype):
    import torch
    from paper_2102_08463_amd import Batch, Plan
    note(f"batch small {prec} {eps} type{ntype}")
    n_modes = [(24, 20), (1, 1), (33, 17), (64, 64), (9, 40)]
    n_points = [5000, 77, 0, 12000, 3001]
    kinds = ["uniform", "uniform", "uniform", "cluster", "uniform"]
    pts, tens, cdt = _batch_inputs(n_modes, n_points, kinds, prec, seed=3)
    rng = np.random.default_rng(5)
    b = Batch(ntype, n_modes, n_points, eps=eps, dtype=torch.complex64 if prec == "f32" else torch.complex128,
              binsize=[(8, 8), (32, 32), (16, 32), (32, 32), (16, 16)], msub=[256, 64, 1024, 500, 2048])
    b.setpts(*tens)
    if ntype == 1:
        cs = [(rng.standard_normal(M) + 1j * rng.standard_normal(M)).astype(cdt) for M in n_points]
        out = b.execute(torch.from_numpy(np.concatenate(cs)).cuda())
        fs = b.split_modes(out)
        for t in range(len(n_modes)):
            got = fs[t].cpu().numpy()
            ref = direct.type1(tuple(a.astype(np.float64) for a in pts[t]), cs[t].astype(np.complex128),
                               n_modes[t], iflag=-1)
            if n_points[t] == 0:
                assert np.count_nonzero(got) == 0
            else:
                assert rel_l2(got, ref) <= 10 * eps, t
            # the same transform on its own plan
            if n_points[t]:
                with Plan(1, n_modes[t], 1, eps, -1, dtype=b.dtype, binsize=None) as p:
                    p.setpts(*[torch.from_numpy(a).cuda() for a in pts[t]])
                    single = p.execute(torch.from_numpy(cs[t]).cuda()).cpu().numpy()
                assert rel_l2(got, single) <= 2 * eps
    else:
        fs = [(rng.standard_normal(nm[::-1]) + 1j * rng.standard_normal(nm[::-1])).astype(cdt) for nm in n_modes]
        out = b.execute(torch.from_numpy(np.concatenate([f.ravel() for f in fs])).cuda()).cpu().numpy()
        off = 0
        for t in range(len(n_modes)):
            got = out[off:off + n_points[t]]
            off += n_points[t]
            if n_points[t] == 0:
                continue
            ref = direct.type2(tuple(a.astype(np.float64) for a in pts[t]), fs[t].astype(np.complex128), iflag=+1)
            assert rel_l2(got, ref) <= 10 * eps, t
    b.destroy()


@pytest.mark.parametrize("kind", ["uniform", "cluster", "radial"])
def test_batch_64_fullsize(kind):
    """64 2D transforms, modes uniform in {64..512}^2, M lognormal (median 2e5,
    1e4..4e6), eps 1e-6 fp32, type 1 then type 2; 4 transforms checked at
    sampled modes / points against the exact sums."""
    import torch
    from paper_2102_08463_amd import Batch
    note(f"batch 64 {kind}")
    n_modes, n_points = workloads.batch_descriptors(64)
    kinds = [kind] * 64
    pts, tens, cdt = _batch_inputs(n_modes, n_points, kinds, "f32", seed=100)
    rng = np.random.default_rng(9)
    cs = [(rng.standard_normal(M) + 1j * rng.standard_normal(M)).astype(cdt) for M in n_points]
    b1 = Batch(1, n_modes, n_points, eps=1e-6)
    b1.setpts(*tens)
    fs = b1.split_modes(b1.execute(torch.from_numpy(np.concatenate(cs)).cuda()))
    check = [int(i) for i in np.argsort(n_points)[[0, 20, 40, 63]]]
    for t in check:
        kk = tuple(np.sort(rng.choice(np.arange(-(N // 2), N - N // 2), size=24, replace=False)) for N in n_modes[t])
        ref = direct.type1(tuple(a.astype(np.float64) for a in pts[t]), cs[t].astype(np.complex128),
                           n_modes[t], iflag=-1, kk=kk)
        got = fs[t].cpu().numpy()[np.ix_(kk[1] + n_modes[t][1] // 2, kk[0] + n_modes[t][0] // 2)]
        assert rel_l2(got, ref) <= 1e-5, t
    b1.destroy()
    b2 = Batch(2, n_modes, n_points, eps=1e-6)
    b2.setpts(*tens)
    fm = [(rng.standard_normal(nm[::-1]) + 1j * rng.standard_normal(nm[::-1])).astype(cdt) for nm in n_modes]
    c = b2.execute(torch.from_numpy(np.concatenate([f.ravel() for f in fm])).cuda()).cpu().numpy()
    offs = np.concatenate([[0], np.cumsum(n_points)])
    for t in check:
        idx = rng.choice(n_points[t], size=min(500, n_points[t]), replace=False)
        ref = direct.type2(tuple(a.astype(np.float64) for a in pts[t]), fm[t].astype(np.complex128),
                           iflag=+1, idx=idx)
        got = c[offs[t]:offs[t + 1]][idx]
        assert rel_l2(got, ref) <= 1e-5, t
    b2.destroy()


@pytest.mark.parametrize("prec,eps", [("f32", 1e-5), ("f64", 1e-8)])
@pytest.mark.parametrize("ntype", [1, 2])
def test_small_mixed_batch_3d(prec, eps, ntype):
    """3D transforms of different sizes, bins and msub in one batch (four
    classes of equal bins and msub, one transform without points): each
    within 10 eps of its exact sums."""
    import torch
    from paper_2102_08463_amd import Batch
    note(f"batch small 3d {prec} {eps} type{ntype}")
    n_modes = [(12, 10, 14), (20, 16, 8), (9, 9, 9), (16, 16, 16), (6, 20, 10)]
    n_points = [3000, 2500, 0, 4000, 1200]
    kinds = ["uniform", "cluster", "uniform", "gaussian", "uniform"]
    pts, tens, cdt = _batch_inputs(n_modes, n_points, kinds, prec, seed=21)
    rng = np.random.default_rng(6)
    b = Batch(ntype, n_modes, n_points, eps=eps,
              dtype=torch.complex64 if prec == "f32" else torch.complex128,
              binsize=[(8, 8, 8), (16, 8, 4), (8, 8, 8), (16, 8, 8), (16, 8, 4)],
              msub=[256, 1024, 256, 512, 1024])
    b.setpts(*tens)
    if ntype == 1:
        cs = [(rng.standard_normal(M) + 1j * rng.standard_normal(M)).astype(cdt) for M in n_points]
        fs = b.split_modes(b.execute(torch.from_numpy(np.concatenate(cs)).cuda()))
        for t in range(len(n_modes)):
            got = fs[t].cpu().numpy()
            if n_points[t] == 0:
                assert np.count_nonzero(got) == 0
                continue
            ref = direct.type1(tuple(a.astype(np.float64) for a in pts[t]),
                               cs[t].astype(np.complex128), n_modes[t], iflag=-1)
            assert rel_l2(got, ref) <= 10 * eps, t
    else:
        fm = [(rng.standard_normal(nm[::-1]) + 1j * rng.standard_normal(nm[::-1])).astype(cdt)
              for nm in n_modes]
        c = b.execute(torch.from_numpy(np.concatenate([f.ravel() for f in fm])).cuda()).cpu().numpy()
        off = 0
        for t in range(len(n_modes)):
            got = c[off:off + n_points[t]]
            off += n_points[t]
            if n_points[t] == 0:
                continue
            ref = direct.type2(tuple(a.astype(np.float64) for a in pts[t]),
                               fm[t].astype(np.complex128), iflag=+1)
            assert rel_l2(got, ref) <= 10 * eps, t
    b.destroy()


@pytest.mark.parametrize("typ", [1, 2])
@pytest.mark.parametrize("modes", [
    [(20, 12)],                                        # one transform: the plan's bins
    [(5, 7), (300, 243), (64, 64), (16, 16)],          # bins wider than a grid
    [(500, 400), (512, 512), (24, 30)],                # 32 x 32 throughout
    [(24, 20), (30, 26)],                              # halved to the narrowest
])
def test_default_bins_shared_by_the_batch(typ, modes):
    """Whatever default bins a batch takes, each transform is what its own plan
    computes, up to the rounding of either (both within 10 eps of the sums)."""
    import torch
    import workloads
    from paper_2102_08463_amd import Batch, Plan
    note(f"batch default bins {typ} {modes}")
    eps = 1e-5
    M = [3000 + 977 * t for t in range(len(modes))]
    pts = [workloads.uniform(m, 2, seed=60 + t) for t, m in enumerate(M)]
    x = [torch.from_numpy(np.concatenate([p[d] for p in pts]).astype(np.float32)).cuda()
         for d in range(2)]
    n_in = sum(M) if typ == 1 else sum(a * b for a, b in modes)
    data = torch.from_numpy(workloads.strengths(n_in, seed=61).astype(np.complex64)).cuda()
    with Batch(typ, modes, M, eps=eps) as b:
        b.setpts(*x)
        out = b.execute(data)
    at = kat = 0
    for md, m in zip(modes, M):
        k = md[0] * md[1]
        d = data[at:at + m] if typ == 1 else data[kat:kat + k]
        with Plan(typ, md, eps=eps) as p:
            p.setpts(*[v[at:at + m].contiguous() for v in x])
            got = p.execute(d.contiguous()).reshape(-1)
        want = out[kat:kat + k] if typ == 1 else out[at:at + m]
        assert float(torch.linalg.norm(got - want) / torch.linalg.norm(got)) <= 20 * eps
        at, kat = at + m, kat + k
