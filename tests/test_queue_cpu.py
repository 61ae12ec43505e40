"""Which launches of the matrix-core kernels take a work counter, and that their LDS
fits: the library's host code with a stand-in for the HIP runtime."""
from tests import host_shim


def test_interp_beside_another_takes_no_counter(tmp_path):
    host_shim.run(tmp_path, """
    for elsewhere in (False, True):
        h = plan(2, (30, 30, 30), eps=1e-9, prec=1, iflag=1, stream=0x51000)
        assert setpts(h, 5000, 3) == 0
        if elsewhere:
            fake.fake_capture(0x51000)
        fake.fake_clear()
        assert lib.mnufft_interp(h, P[3], P[4]) == 0
        assert count(QUEUE) == (0 if elsewhere else 1)
        fake.fake_capture(None)
        fake.fake_clear()
        assert lib.mnufft_interp(h, P[3], P[4]) == 0
        assert count(QUEUE) == (0 if elsewhere else 1)
        fake.fake_clear()
        assert lib.mnufft_execute(h, P[3], P[4]) == 0    # on the plan's grid: with it
        assert count(QUEUE) == 1
        lib.mnufft_destroy(h)
    """)


def test_largest_bins_fit_with_the_static_lds(tmp_path):
    """Bins whose tile and staged points fill the 160 KB to the last byte (9207 cells
    at w = 8) leave no room for the kernel's static LDS: they take the other kernel,
    as every bin that was accepted before runs."""
    host_shim.run(tmp_path, """
    for bins in ((23, 19, 3), (19, 23, 3), (3, 19, 23), (24, 16, 4), (16, 8, 8)):
        h = plan(1, (40, 40, 40), eps=1e-7, prec=1, binsize=(ci * 3)(*bins))
        assert setpts(h, 5000, 3) == 0
        assert lib.mnufft_execute(h, P[3], P[4]) == 0
        assert lib.mnufft_execute_adjoint(h, P[3], P[4]) == 0
        assert count(OVERRUN) == 0, bins
        lib.mnufft_destroy(h)
    """)
