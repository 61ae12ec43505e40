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
