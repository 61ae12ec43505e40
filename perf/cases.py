"""Timed workloads of the library, through its Python entry points.

Each case is one pass of a program that uses the library.  ``do`` says what the
pass consists of:

  step    set the points, transform, and apply the adjoint on the same points:
          a solver whose points change every iteration
  points  set the points and transform once (slicing / merging steps)
  apply   transform and adjoint on points set beforehand (an iterative solver
          with fixed points), for one or several vectors
  once    one transform on points set beforehand
  batch   many 2D transforms of uneven size through ``Batch``
  type3   nonuniform points to nonuniform frequencies
  grad    a differentiable type 2 forward and backward, as a training step

Inputs are drawn on the GPU from the seed.  ``exact`` evaluates the defining
sums in double precision with plain torch.
"""
import math

import torch

from paper_2102_08463_amd import Batch, Plan
from paper_2102_08463_amd import autograd

PI = math.pi
TWO_PI = 2.0 * math.pi
REAL = {"f32": torch.float32, "f64": torch.float64}
CPLX = {"f32": torch.complex64, "f64": torch.complex128}


def _case(name, do, type_, modes, M, eps, prec, points, ntrans=1, sigma=2.0, K=0):
    n = list(modes) + [0] * (3 - len(modes))
    c = {"do": do, "type": type_, "dim": len(modes), "n1": n[0], "n2": n[1], "n3": n[2],
         "M": M, "K": K, "eps": eps, "prec": prec, "points": points, "ntrans": ntrans,
         "sigma": sigma}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a small image: launches and latency are all there is
        _case("2d 64 step", "step", 1, (64, 64), 100_000, 1e-5, "f32", "uniform"),
        # the benchmark's default workload
        _case("2d 1024 step", "step", 1, (1024, 1024), 10_000_000, 1e-5, "f32", "uniform"),
        # all points in a small square of the same grid, points kept
        _case("2d 1024 cluster type 1", "once", 1, (1024, 1024), 10_000_000, 1e-5, "f32",
              "cluster"),
        # tight tolerance in double precision, odd sizes
        _case("2d 999x1000 f64 step", "step", 1, (999, 1000), 3_000_001, 1e-9, "f64", "uniform"),
        # the 3D benchmark workload
        _case("3d 128 step", "step", 1, (128, 128, 128), 1 << 24, 1e-5, "f32", "uniform"),
        # the slicing step of a reconstruction: 3D type 2 on random Ewald-sphere caps
        _case("3d 41 f64 slicing", "points", 2, (41, 41, 41), 1000 * 32 * 32, 1e-12, "f64",
              "caps32"),
        # its merging step: 3D type 1, many points on a small grid
        _case("3d 81 f64 merging", "points", 1, (81, 81, 81), 1000 * 128 * 128, 1e-12, "f64",
              "caps128"),
        # radial sampling with eight receivers, forward and adjoint of a solver
        _case("2d 256 radial x8 apply", "apply", 2, (256, 256), 256 * 512, 1e-6, "f32",
              "radial", ntrans=8),
        # the batched workload: 64 transforms, modes in [64, 512]^2, uneven M
        _case("2d batch of 64", "batch", 1, (64, 512), 200_000, 1e-6, "f32", "uniform",
              ntrans=64),
        # nonuniform to nonuniform
        _case("2d type 3", "type3", 3, (512, 512), 1_000_000, 1e-5, "f32", "uniform",
              K=600_000),
        # training step through a 3D type 2 on a stack of spirals
        _case("3d 64 spirals gradient", "grad", 2, (64, 64, 64), 4_000_000, 1e-5, "f32",
              "spirals"),
        # a long 1D signal with jittered samples
        _case("1d 2^20 step", "step", 1, (1 << 20,), 10_000_000, 1e-5, "f32", "uniform"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["step", "step", "points", "points", "apply", "once", "batch", "type3",
                     "grad"])
    prec = rng.choice(["f32", "f32", "f64"])
    eps = 10.0 ** -(rng.randint(2, 6) if prec == "f32" else rng.randint(7, 12))
    sigma = 2.0
    if do == "batch":
        T = _log(rng, 4, 64)
        return _case(None, do, rng.choice([1, 2]), (_log(rng, 24, 64), _log(rng, 128, 512)),
                     _log(rng, 5_000, 200_000), eps, prec,
                     rng.choice(["uniform", "cluster", "radial"]), ntrans=T)
    dim = rng.choice([2, 2, 3, 3, 1]) if do != "type3" else rng.choice([2, 2, 3])
    lo, hi = {1: (200, 1 << 20), 2: (40, 1024), 3: (16, 128)}[dim]
    if do == "type3":
        hi = {2: 400, 3: 40}[dim]
    modes = tuple(_log(rng, lo, hi) for _ in range(dim))
    # what a pass may cost: wide double precision kernels take fewer points
    top = 10_000_000 if prec == "f32" else (4_000_000 if dim < 3 else 2_000_000)
    kinds = {1: ["uniform", "gaussian"], 2: ["uniform", "cluster", "gaussian", "radial"],
             3: ["uniform", "gaussian", "spirals", "caps32"]}[dim]
    points = rng.choice(kinds)
    T, K = 1, 0
    if do in ("apply", "once") and rng.random() < 0.5:
        T = rng.randint(2, 12)
        top //= 16
    if do == "type3":
        top, points, K = 600_000, "uniform", _log(rng, 10_000, 600_000)
    elif do != "grad" and rng.random() < 0.2:
        sigma = rng.choice([1.25, 1.5])
    M = _log(rng, 10_000, top)
    if points == "caps32":
        M = max(1, M // 1024) * 1024
    type_ = {"type3": 3, "grad": 2}.get(do) or rng.choice([1, 2])
    return _case(None, do, type_, modes, M, eps, prec, points, ntrans=T, sigma=sigma, K=K)


# ---- inputs -----------------------------------------------------------------
def _wrap(a):
    return torch.remainder(a + PI, TWO_PI) - PI


def _points(kind, M, dim, g):
    """dim float64 tensors of M coordinates in [-pi, pi)."""
    def u(*shape):
        return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64)

    if kind == "uniform":
        return list(-PI + TWO_PI * u(dim, M))
    if kind == "cluster":    # a square of side 2 pi / 64 at the origin
        return list(TWO_PI / 64 * u(dim, M))
    if kind == "gaussian":
        return list(_wrap(0.1 * normal(dim, M)))
    if kind == "radial":     # spokes through the origin, turned by a random angle
        spokes = 256 if M >= 65536 else 64
        j = torch.arange(M, device="cuda", dtype=torch.float64)
        per = -(-M // spokes)
        s = torch.floor(j / per)
        r = -PI + TWO_PI * (j - s * per + 0.5) / per
        th = PI * s / spokes + TWO_PI * u(1)
        return [_wrap(r * torch.cos(th)), _wrap(r * torch.sin(th))]
    if kind == "spirals":    # planes of Archimedean spirals with jitter
        planes, turns = 64, 32
        j = torch.arange(M, device="cuda", dtype=torch.float64)
        per = -(-M // planes)
        p = torch.floor(j / per)
        t = (j - p * per + 0.5) / per
        zp = -PI + TWO_PI * (p + 0.5) / planes
        x = torch.stack([PI * t * torch.cos(TWO_PI * turns * t),
                         PI * t * torch.sin(TWO_PI * turns * t), zp])
        return list(_wrap(x + 1e-3 * normal(3, M)))
    side = int(kind[4:])     # caps<side>: randomly turned Ewald-sphere caps
    n = M // (side * side)
    t = 0.65 * PI * (-1 + 2 * (torch.arange(side, device="cuda", dtype=torch.float64) + 0.5) / side)
    a, b = (v.reshape(-1) for v in torch.meshgrid(t, t, indexing="xy"))
    cap = torch.stack([a, b, TWO_PI - torch.sqrt(TWO_PI ** 2 - a * a - b * b)])
    q = normal(4, n)
    w, x, y, z = q / torch.linalg.norm(q, dim=0)
    rows = [[1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w)],
            [2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w)],
            [2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)]]
    return [_wrap(sum(r[k][:, None] * cap[k][None, :] for k in range(3)).reshape(-1))
            for r in rows]


def _modes(case):
    return tuple(case["n%d" % (d + 1)] for d in range(case["dim"]))


def _batch_sizes(case, seed):
    """Mode counts uniform in [n1, n2]^2, point counts lognormal about M: the
    sizes belong to the case, not to the seed's values."""
    g = torch.Generator()
    g.manual_seed(7)
    T = case["ntrans"]
    n = torch.randint(case["n1"], case["n2"] + 1, (T, 2), generator=g)
    m = torch.exp(math.log(case["M"]) + torch.randn(T, generator=g, dtype=torch.float64))
    lo, hi = case["M"] / 20, case["M"] * 20
    return ([(int(a), int(b)) for a, b in n],
            [int(v) for v in torch.clamp(torch.round(m), lo, hi)])


def _inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    rt, dim, T = REAL[case["prec"]], case["dim"], case["ntrans"]

    def values(*shape):
        v = torch.randn(*shape, 2, generator=g, device="cuda", dtype=rt)
        return torch.view_as_complex(v)

    if case["do"] == "batch":
        modes, npts = _batch_sizes(case, seed)
        per = [_points(case["points"], m, 2, g) for m in npts]
        x = [torch.cat([p[d] for p in per]).to(rt) for d in range(2)]
        n = sum(npts) if case["type"] == 1 else sum(a * b for a, b in modes)
        return {"x": x, "c": values(n), "modes": modes, "npts": npts}
    x = [a.to(rt).contiguous() for a in _points(case["points"], case["M"], dim, g)]
    lead = (T,) if T > 1 else ()
    d = {"x": x}
    if case["do"] == "type3":
        d["s"] = [(case["n%d" % (i + 1)] * (torch.rand(case["K"], generator=g, device="cuda",
                                                       dtype=torch.float64) * 2 - 1)).to(rt)
                  for i in range(dim)]
        d["c"] = values(*lead, case["M"])
        return d
    d["c"] = values(*lead, case["M"])
    d["f"] = values(*lead, *_modes(case)[::-1])
    return d


# ---- one pass -----------------------------------------------------------------
def prepare(case, seed):
    st = _inputs(case, seed)
    st["case"] = case
    kw = {"eps": case["eps"], "dtype": CPLX[case["prec"]]}
    do = case["do"]
    if do == "batch":
        st["plan"] = Batch(case["type"], st["modes"], st["npts"], **kw)
    elif do == "type3":
        st["plan"] = Plan(3, case["dim"], case["ntrans"], **kw)
    elif do != "grad":
        st["plan"] = Plan(case["type"], _modes(case), case["ntrans"], upsampfac=case["sigma"],
                          **kw)
        if do in ("apply", "once"):
            st["plan"].setpts(*st["x"])
    return st


def run(st):
    case = st["case"]
    do = case["do"]
    if do == "grad":
        f = st["f"].detach().requires_grad_()
        x = [a.detach().requires_grad_() for a in st["x"]]
        c = autograd.nufft_type2(x, f, eps=case["eps"])
        grads = torch.autograd.grad(c, [f] + x, grad_outputs=st["c"])
        return [c.detach()] + list(grads)
    plan = st["plan"]
    if do == "batch":
        plan.setpts(*st["x"])
        return plan.execute(st["c"])
    if do == "type3":
        dim = case["dim"]
        plan.setpts(*st["x"], *([None] * (3 - dim)), *st["s"])
        return plan.execute(st["c"])
    if do in ("step", "points"):
        plan.setpts(*st["x"])
    fwd, adj = ("c", "f") if case["type"] == 1 else ("f", "c")
    out = [plan.execute(st[fwd])]
    if do in ("step", "apply"):
        out.append(plan.execute_adjoint(st[adj]))
    return out


# ---- what a pass cannot do without ------------------------------------------
def _width(case):
    if case["sigma"] == 2.0:
        return max(2, math.ceil(math.log10(1.0 / case["eps"]) - 1e-9) + 1)
    return math.ceil(math.log(1.0 / case["eps"]) / (PI * math.sqrt(1.0 - 1.0 / case["sigma"])))


def work(case):
    rb = 4 if case["prec"] == "f32" else 8
    dim, w, T, do = case["dim"], _width(case), case["ntrans"], case["do"]

    def fft(modes):
        n = 1.0
        for m in modes:
            n *= case["sigma"] * m
        return 5.0 * n * math.log2(max(n, 2.0))

    if do == "batch":
        modes, npts = _batch_sizes(case, 0)
        M, N = sum(npts), sum(a * b for a, b in modes)
        return {"bytes": M * rb * 4 + N * rb * 2,
                "flops": M * 4.0 * w ** 2 + sum(fft(m) for m in modes)}
    M, modes = case["M"], _modes(case)
    if do == "type3":
        K, box = case["K"], [4 * n + w + 1 for n in modes]
        return {"bytes": (M + K) * rb * (dim + 2 * T),
                "flops": T * ((M + K) * 4.0 * w ** dim + fft(box))}
    N = math.prod(modes)
    vec = T * (M + N) * rb * 2        # a transform reads one side and writes the other
    one = T * (M * 4.0 * w ** dim + fft(modes))
    pts = M * rb * dim
    if do == "grad":                  # values, adjoint and dim position gradients
        return {"bytes": pts * 2 + vec * 2, "flops": one * (2 + dim)}
    n = 2 if do in ("step", "apply") else 1
    return {"bytes": (pts if do in ("step", "points") else 0) + n * vec, "flops": n * one}


# ---- the defining sums in 64 bits ---------------------------------------------
def _phases(x, N, sign):
    k = torch.arange(N, device="cuda", dtype=torch.float64) - N // 2
    return torch.polar(torch.ones((), device="cuda", dtype=torch.float64),
                       (sign * x.double())[:, None] * k[None, :])


def _split(x, modes, sign):
    """Two factors per point whose outer product holds exp(i sign k.x) over the
    modes, (M, left) and (M, N1), k1 fastest."""
    if len(modes) == 1:   # k = k_lo + 1024 k_hi
        return None
    left = _phases(x[1], modes[1], sign)
    if len(modes) == 3:
        e3 = _phases(x[2], modes[2], sign)
        left = (e3[:, :, None] * left[:, None, :]).reshape(x[0].shape[0], -1)
    return left, _phases(x[0], modes[0], sign)


def _split1(x, N, sign, width=1024):
    """The same for one dimension: k = -(N // 2) + lo + width hi."""
    hi = -(-N // width)
    one = torch.ones((), device="cuda", dtype=torch.float64)
    xd = sign * x.double()
    lo = torch.arange(width, device="cuda", dtype=torch.float64) - N // 2
    up = torch.arange(hi, device="cuda", dtype=torch.float64) * width
    return torch.polar(one, xd[:, None] * up[None, :]), torch.polar(one, xd[:, None] * lo[None, :])


def _chunks(x, modes, sign):
    left = math.prod(modes[1:]) if len(modes) > 1 else -(-modes[0] // 1024)
    step = max(256, min(65536, (1 << 27) // max(left, modes[0] if len(modes) > 1 else 1024)))
    for a in range(0, x[0].shape[0], step):
        xs = [v[a:a + step] for v in x]
        yield slice(a, a + step), (_split1(xs[0], modes[0], sign) if len(modes) == 1
                                   else _split(xs, modes, sign))


def _type1(x, c, modes, sign):
    """c (T, M) -> (T, ..., N2, N1)."""
    out = None
    for sl, (A, B) in _chunks(x, modes, sign):
        # (left, M) (M, N1), once per vector
        got = torch.stack([torch.mm((A * v[sl].to(torch.complex128)[:, None]).t().contiguous(), B)
                           for v in c])
        out = got if out is None else out + got
    if len(modes) == 1:
        return out.reshape(len(c), -1)[:, :modes[0]]
    return out.reshape((len(c),) + tuple(modes[::-1]))


def _type2(x, f, modes, sign):
    """f (T, ..., N2, N1) -> (T, M)."""
    T = f.shape[0]
    g = f.to(torch.complex128).reshape(T, -1)
    if len(modes) == 1:
        hi = -(-modes[0] // 1024)
        g = torch.nn.functional.pad(g, (0, hi * 1024 - modes[0])).reshape(T, hi, 1024)
    else:
        g = g.reshape(T, -1, modes[0])
    out = torch.empty(T, x[0].shape[0], device="cuda", dtype=torch.complex128)
    for sl, (A, B) in _chunks(x, modes, sign):
        for t in range(T):
            out[t, sl] = (torch.mm(A, g[t]) * B).sum(dim=1)
    return out


def exact(case, seed):
    do, T, dim = case["do"], case["ntrans"], case["dim"]
    if do == "batch":
        d = _inputs(case, seed)
        outs, at, kat = [], 0, 0
        for n, m in zip(d["modes"], d["npts"]):
            x = [v[at:at + m] for v in d["x"]]
            k = n[0] * n[1]
            if case["type"] == 1:
                outs.append(_type1(x, d["c"][None, at:at + m], n, -1).reshape(-1))
            else:
                outs.append(_type2(x, d["c"][None, kat:kat + k].reshape(1, n[1], n[0]), n,
                                   1).reshape(-1))
            at, kat = at + m, kat + k
        return torch.cat(outs)
    if do == "type3":
        if case["M"] * case["K"] * T > 7e11:
            return None
        d = _inputs(case, seed)
        X = torch.stack([v.double() for v in d["x"]], dim=1)
        S = torch.stack([v.double() for v in d["s"]])
        c = d["c"].to(torch.complex128).reshape(T, -1)
        out = torch.zeros(T, case["K"], device="cuda", dtype=torch.complex128)
        step = max(1, (1 << 28) // case["K"])
        for a in range(0, case["M"], step):
            ph = torch.mm(X[a:a + step], S)
            cc = c[:, a:a + step]
            e, s = torch.cos(ph), torch.sin(ph)
            out += torch.complex(cc.real @ e + cc.imag @ s, cc.imag @ e - cc.real @ s)
        return out if T > 1 else out[0]
    modes = _modes(case)
    sums = {"grad": 2 + dim, "step": 2, "apply": 2}.get(do, 1) * T
    if sums * float(case["M"]) * math.prod(modes) > 8e13:
        return None
    d = _inputs(case, seed)
    c = d["c"].reshape(T, -1)
    f = d["f"].reshape((T,) + modes[::-1])
    if do == "grad":
        v = _type2(d["x"], f, modes, 1)
        out = [v[0], _type1(d["x"], c, modes, -1)[0]]
        for i in range(dim):
            k = torch.arange(modes[i], device="cuda", dtype=torch.float64) - modes[i] // 2
            shape = [1] * (dim + 1)
            shape[dim - i] = modes[i]
            dv = _type2(d["x"], f.to(torch.complex128) * (1j * k.reshape(shape)), modes, 1)
            out.append((c.to(torch.complex128).conj() * dv).real[0])
        return out
    sign1, sign2 = (-1, 1)

    def shaped(v):
        return v if T > 1 else v[0]

    one = lambda: shaped(_type1(d["x"], c, modes, sign1))  # noqa: E731
    two = lambda: shaped(_type2(d["x"], f, modes, sign2))  # noqa: E731
    order = [one, two] if case["type"] == 1 else [two, one]
    return [fn() for fn in (order if do in ("step", "apply") else order[:1])]
