"""Point buffers of a plan hold every smaller point set too: the library's host
code with a stand-in for the HIP runtime, which checks what the sort's kernels
are given against the blocks they write."""
import pytest

from tests import host_shim


@pytest.mark.parametrize("dim,prec", [(1, 0), (2, 0), (3, 0), (2, 1), (3, 1)])
@pytest.mark.parametrize("method", [0, 1])
def test_fewer_points_on_a_plan(tmp_path, dim, prec, method):
    host_shim.run(tmp_path, f"""
    dim, prec, method = {dim}, {prec}, {method}
    MI = 1 << 20
    firsts = [MI - 1, MI, MI + 1, 1_100_000, 1_500_000, 4 * MI - 4096, 4 * MI, 4 * MI + 1, 5 * MI]
    thens = [MI, MI - 1, 1_000_000, 900_000, 263_000, 262_145, 262_144, 262_143, 65_537, 2049, 1, 0]
    modes = [(4096,), (96, 90), (20, 18, 24)][dim - 1]
    for first in firsts:
        h = plan(1, modes, eps=1e-5 if prec == 0 else 1e-9, prec=prec, method=method)
        for m in [first] + [t for t in thens if t <= first] + [first]:
            assert setpts(h, m, dim) == 0
            assert count(OVERRUN) == 0, (first, m)
        lib.mnufft_destroy(h)
    """)


def test_fewer_points_in_type3(tmp_path):
    host_shim.run(tmp_path, """
    for first in ((1 << 20) + 1, 1_100_000, 4_000_000):
        h = plan(3, (1, 1))
        for m, k in ((first, first), (1_000_000, 1 << 20), (1 << 20, 900_000), (5, 1)):
            assert lib.mnufft_setpts3(h, m, P[0], P[1], None, k, P[2], P[3], None) == 0
            assert count(OVERRUN) == 0, (first, m, k)
        lib.mnufft_destroy(h)
    """)
