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
