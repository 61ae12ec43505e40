"""Runs the library's host code without a GPU, in a process of its own where
tests/native/fake_hip.c takes the place of the HIP runtime: ``run(code)``
executes ``code`` there with ``lib`` (the library), ``fake`` (the stand-in's
own functions) and the helpers below."""
import os
import subprocess
import sys
import textwrap

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
vp, i64, ci, dbl = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_double
for f in (fake.fake_count, fake.fake_live):
    f.restype = ctypes.c_longlong
fake.fake_capacity.argtypes = [ctypes.c_longlong]
fake.fake_capture.argtypes = fake.fake_stream_gone.argtypes = [vp]
MALLOC, FREE, STREAM_SYNC, DEVICE_SYNC, LAUNCH, OVERRUN, SYNC_DEV, QUEUE = range(8)
count, live = fake.fake_count, fake.fake_live
P = [vp((1 << 40) + (k << 36)) for k in range(8)]   # addresses of a caller's buffers
lib.mnufft_makeplan.argtypes = [ci, ci, vp, ci, i64, dbl, ci, vp, vp]
lib.mnufft_setpts.argtypes = [vp, i64, vp, vp, vp]
lib.mnufft_setpts3.argtypes = [vp, i64, vp, vp, vp, i64, vp, vp, vp]
lib.mnufft_batch_makeplan.argtypes = [ci, ci, ci, vp, vp, ci, dbl, ci, vp, vp, vp, vp]
for name in ("execute", "execute_adjoint", "execute_sorted", "spread", "interp", "batch_execute"):
    getattr(lib, "mnufft_" + name).argtypes = [vp, vp, vp]
lib.mnufft_interp_grad.argtypes = [vp] * 6
lib.mnufft_get_sort.argtypes = lib.mnufft_get_subproblems.argtypes = [vp] * 3
lib.mnufft_batch_setpts.argtypes = [vp] * 4
lib.mnufft_set_stream.argtypes = [vp, vp]
lib.mnufft_destroy.argtypes = lib.mnufft_batch_destroy.argtypes = [vp]

class Opts(ctypes.Structure):
    _fields_ = [("method", ci), ("binsize", ci * 3), ("msub", ci), ("validate_pts", ci),
                ("device", ci), ("stream", vp), ("upsampfac", dbl), ("tune", ci),
                ("reserved", ci * 5)]

def opts(**kw):
    o = Opts()
    lib.mnufft_default_opts(ctypes.byref(o))
    for k, v in kw.items():
        setattr(o, k, v)
    return o

def plan(type_, modes, nt=1, eps=1e-5, prec=0, iflag=-1, ok=True, **kw):
    h = vp()
    n = (i64 * 3)(*(list(modes) + [1] * (3 - len(modes))))
    o = opts(**kw)
    rc = lib.mnufft_makeplan(type_, len(modes), n, iflag, nt, eps, prec, ctypes.byref(o),
                             ctypes.byref(h))
    assert rc >= 0 or not ok, rc
    return h if ok else (rc, h)

def batch(type_, modes, npts, eps=1e-5, prec=0, iflag=-1, **kw):
    h, T = vp(), len(modes)
    n = (i64 * (3 * T))(*[v for m in modes for v in list(m) + [1] * (3 - len(m))])
    o = opts(**kw)
    rc = lib.mnufft_batch_makeplan(type_, len(modes[0]), T, n, (i64 * T)(*npts), iflag, eps, prec,
                                   None, None, ctypes.byref(o), ctypes.byref(h))
    assert rc >= 0, rc
    return h

def setpts(h, M, dim):
    return lib.mnufft_setpts(h, M, P[0], P[1] if dim > 1 else None, P[2] if dim > 2 else None)
"""


def build(folder):
    """The stand-in as a shared library in ``folder``."""
    so = os.path.join(str(folder), "libfake_hip.so")
    if not os.path.exists(so):
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so,
                        os.path.join(ROOT, "tests", "native", "fake_hip.c")], check=True)
    return so


def run(folder, code):
    """Runs ``code``; what it prints.  Fails with its output if it fails."""
    lib = os.path.join(ROOT, "paper_2102_08463_amd", "libmnufft.so")
    r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(code), build(folder), lib],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-3000:]
    return r.stdout
