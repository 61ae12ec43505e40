"""Allocations that fail: the library's host code with a stand-in for the HIP
runtime whose memory runs out."""
import pytest

from tests import host_shim


@pytest.mark.parametrize("dim,prec,method", [(1, 0, 0), (2, 0, 0), (2, 1, 0), (3, 0, 0), (3, 1, 0),
                                             (2, 0, 1), (3, 0, 2)])
def test_failed_setpts_leaves_nothing_behind(tmp_path, dim, prec, method):
    """Whichever of its allocations fails: the call says so, the plan still takes
    points, and all its memory comes back."""
    host_shim.run(tmp_path, f"""
    dim, prec, method = {dim}, {prec}, {method}
    modes = (40, 44, 36)[:dim]
    h = plan(1, modes, eps=1e-9 if prec else 1e-5, prec=prec, method=method)
    base = live()
    assert setpts(h, 200000, dim) == 0
    most = live() - base
    lib.mnufft_destroy(h)
    failed = 0
    for part in range(40):
        assert lib.mnufft_release_memory() == 0 and live() == 0, part
        h = plan(1, modes, eps=1e-9 if prec else 1e-5, prec=prec, method=method)
        fake.fake_capacity(live() + most * part // 40)
        rc = setpts(h, 200000, dim)
        assert rc in (0, -2), rc
        failed += rc == -2
        fake.fake_capacity(-1)
        assert lib.mnufft_execute(h, P[3], P[4]) == (0 if rc == 0 else -5)
        assert setpts(h, 1000, dim) == 0
        assert lib.mnufft_execute(h, P[3], P[4]) == 0
        assert lib.mnufft_destroy(h) == 0
    assert failed > 20
    """)


def test_tiles_of_stacked_transforms_where_memory_is_short(tmp_path):
    """What fits with the tiles of one transform is accepted."""
    host_shim.run(tmp_path, """
    class Info(ctypes.Structure):   # (device_bytes alone is read)
        _fields_ = [("pad", ci * 4), ("n", i64 * 6), ("ntransf", i64), ("M", i64), ("w", ci),
                    ("beta", dbl), ("method", ci), ("binsize", ci * 3), ("msub", ci), ("nbins", i64),
                    ("nsub_max", i64), ("device_bytes", i64), ("rest", i64 * 2)]
    def used(h):
        i = Info()
        lib.mnufft_get_info(h, ctypes.byref(i))
        return i.device_bytes
    def points(nt, M):              # bytes of the point set alone
        h = plan(1, (64, 64), nt=nt)
        before = used(h)
        assert setpts(h, M, 2) == 0
        n = used(h) - before
        lib.mnufft_destroy(h)
        return n
    M, nt = 50000, 64
    one, many = points(1, M), points(nt, M)
    assert many > 4 * one
    for room in (one * 5 // 4, one * 2, one * 8):
        lib.mnufft_release_memory()
        h = plan(1, (64, 64), nt=nt)
        fake.fake_capacity(live() + room)
        assert setpts(h, M, 2) == 0, room
        assert lib.mnufft_execute(h, P[3], P[4]) == 0
        fake.fake_capacity(-1)
        lib.mnufft_destroy(h)
    """)


def test_block_that_fits_without_its_rest(tmp_path):
    """Sizes are rounded up so that blocks fit the next plan; where only the asked
    size is left, that is taken."""
    host_shim.run(tmp_path, """
    h = plan(2, (1000, 1000))                   # 2000^2 cells: 32,000,000 bytes, class 33,554,432
    small = live()
    lib.mnufft_destroy(h)
    lib.mnufft_release_memory()
    fake.fake_capacity(small - 33_554_432 + 32_000_000)
    rc, h = plan(2, (1000, 1000), ok=False)
    assert rc == 0
    """)
