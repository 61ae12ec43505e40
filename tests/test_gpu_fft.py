"""The fine-grid FFT with truncation / padding and correction factors in its
passes, against numpy's FFT of the same grid in double precision: every radix,
lengths that need several stages, the two-pass 1D form, stacked transforms."""
import ctypes

import numpy as np
import pytest
import torch

import workloads
from paper_2102_08463_amd import Batch, Plan, lib

pytestmark = pytest.mark.gpu

# modes -> fine lengths: 12, 15 / 90, 2160 / 2048 x 4 / 4320 (24 values a
# thread) / 3D odd sizes / 1D one line, then two passes (8640, 2^17)
CASES = [((5, 7), 1), ((45, 1080), 1), ((1024, 2), 3), ((2160, 3), 1), ((300, 243), 1),
         ((9, 10, 32), 1), ((27, 8, 5), 2), ((64, 40, 50), 1),
         ((6,), 3), ((2048,), 1), ((4099,), 2), ((65536,), 1),
         ((128, 12), 1), ((32, 8, 16), 2), ((3, 5000), 1)]


def _factors(info, d):
    lb = lib.load()
    N, n = info["nmodes"][d], info["nfine"][d]
    out = (ctypes.c_double * N)()
    assert lb.mnufft_correction_factors(N, n, info["w"], info["beta"], out) == 0
    return np.array(out[:])


def _tol(dtype, cells):
    # backward error of a split-radix FFT: a few roundings per level, in the 2-norm
    eps = 2.0 ** -24 if dtype == torch.complex64 else 2.0 ** -53
    return 8 * eps * np.log2(cells)


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("modes,T", CASES)
def test_passes_match_fft(modes, T, dtype):
    dim = len(modes)
    M = 300
    rd = np.float32 if dtype == torch.complex64 else np.float64
    cd = np.complex64 if dtype == torch.complex64 else np.complex128
    pts = [torch.from_numpy(a.astype(rd)).cuda() for a in workloads.uniform(M, dim, seed=3)]
    for isign in (-1, 1):
        with Plan(1, modes, T, 1e-5, isign, dtype=dtype) as p:
            p.setpts(*pts)
            info = p.info()
            c = torch.from_numpy(workloads.strengths((T, M), seed=4).astype(cd)).cuda()
            got = p.execute(c if T > 1 else c[0]).cpu().numpy().reshape((T,) + modes[::-1])
            back = torch.from_numpy(
                workloads.strengths((T,) + modes[::-1], seed=5).astype(cd)).cuda()
            vals = p.execute_adjoint(back if T > 1 else back[0]).cpu().numpy().reshape(T, M)
            grids = [p.spread(c[t].contiguous()).cpu().numpy().astype(np.complex128)
                     for t in range(T)]
            nf = info["nfine"][:dim]
            fac = [_factors(info, d) for d in range(dim)]
            scale = fac[0]
            for d in range(1, dim):
                scale = fac[d].reshape((-1,) + (1,) * d) * scale
            sel = np.ix_(*[(np.arange(modes[d]) - modes[d] // 2) % nf[d]
                           for d in reversed(range(dim))])
            cells = int(np.prod(nf))
            for t in range(T):
                fft = np.fft.fftn if isign < 0 else (lambda a: np.fft.ifftn(a) * a.size)
                want = fft(grids[t])[sel] * scale
                err = np.linalg.norm(got[t] - want) / np.linalg.norm(want)
                assert err <= _tol(dtype, cells), (modes, isign, t, err)
                pad = np.zeros(nf[::-1], dtype=np.complex128)
                pad[sel] = back[t].cpu().numpy().astype(np.complex128) * scale
                inv = np.fft.fftn if isign > 0 else (lambda a: np.fft.ifftn(a) * a.size)
                g = torch.from_numpy(inv(pad).astype(cd)).cuda()
                ref = p.interp(g).cpu().numpy()
                err = np.linalg.norm(vals[t] - ref) / np.linalg.norm(ref)
                assert err <= _tol(dtype, cells), (modes, isign, t, err)


@pytest.mark.parametrize("typ", [1, 2])
def test_batch_passes_match_plans(typ):
    """A batch's single launch per pass gives what each transform's plan gives."""
    modes = [(5, 7), (300, 243), (64, 64), (1000, 9)]
    M = [100, 2000, 1, 500]
    pts = [workloads.uniform(m, 2, seed=i) for i, m in enumerate(M)]
    x = [torch.from_numpy(np.concatenate([p[d] for p in pts]).astype(np.float32)).cuda()
         for d in range(2)]
    n_in = sum(M) if typ == 1 else sum(a * b for a, b in modes)
    data = torch.from_numpy(workloads.strengths(n_in, seed=9).astype(np.complex64)).cuda()
    with Batch(typ, modes, M, eps=1e-5) as b:
        b.setpts(*x)
        out = b.execute(data)
    at = kat = 0
    for md, m in zip(modes, M):
        k = md[0] * md[1]
        with Plan(typ, md, eps=1e-5) as p:
            p.setpts(*[v[at:at + m].contiguous() for v in x])
            d = data[at:at + m] if typ == 1 else data[kat:kat + k]
            got = p.execute(d.contiguous()).reshape(-1)
        want = out[kat:kat + k] if typ == 1 else out[at:at + m]
        err = torch.linalg.norm(got - want) / torch.linalg.norm(want)
        assert err <= 2 * _tol(torch.complex64, 4 * k), (md, float(err))
        at, kat = at + m, kat + k


@pytest.mark.parametrize("sigma,eps,own", [(2.0, 1e-6, True), (1.25, 1e-4, True),
                                           (1.25, 1e-6, False)])
def test_plans_that_amplify_rounding_keep_the_library_fft(sigma, eps, own):
    """3D single precision at 43 and 1550 times amplified rounding: the own
    passes apply the factors themselves, the library's FFT needs the kernel."""
    modes, M = (20, 18, 16), 2000
    pts = [torch.from_numpy(a.astype(np.float32)).cuda()
           for a in workloads.uniform(M, 3, seed=11)]
    f = torch.from_numpy(workloads.strengths(modes[::-1], seed=12).astype(np.complex64)).cuda()
    with Plan(2, modes, 1, eps, -1, upsampfac=sigma) as p:
        p.setpts(*pts)
        p.set_timing(True)
        p.execute(f)
        _, launches = p.timing()["precorrect"]
    assert (launches == 0) == own
