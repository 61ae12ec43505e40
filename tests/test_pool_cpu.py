"""Memory kept from destroyed plans goes back to the system: the library's host
code with a stand-in for the HIP runtime, which counts what is allocated."""
from tests import host_shim


def test_release_memory(tmp_path):
    host_shim.run(tmp_path, """
    for dim in (2, 3):
        h = plan(1, (64, 60, 50)[:dim])
        assert setpts(h, 100000, dim) == 0
        b = batch(1, [(64, 60), (32, 40)], [1000, 500])
        assert lib.mnufft_release_memory() == 0
        used = live()
        assert used > 0
        lib.mnufft_destroy(h)
        lib.mnufft_batch_destroy(b)
        assert live() == used                  # kept for the next plan
        assert lib.mnufft_release_memory() == 0
        assert live() == 0
    """)


def test_old_memory_goes_at_the_next_call(tmp_path):
    """At a call that only allocates, too, and only what is old."""
    host_shim.run(tmp_path, """
    small = plan(1, (16, 16))
    base = live()
    h = plan(1, (256, 256))
    lib.mnufft_destroy(h)
    assert live() > base
    fake.fake_time.argtypes = [dbl]
    fake.fake_time(9.0)
    other = plan(1, (30, 30))
    assert live() > base + (1 << 20)           # the 512 x 512 grid is still there
    fake.fake_time(11.0)
    fake.fake_clear()
    third = plan(1, (33, 35))
    assert count(FREE) > 0
    for p in (small, other, third):
        lib.mnufft_destroy(p)
    held = live()
    fake.fake_time(12.0)
    assert lib.mnufft_release_memory() == 0 and live() == 0 and held > 0
    """)


def test_kept_memory_is_bounded(tmp_path):
    host_shim.run(tmp_path, """
    plans = [plan(1, (2048, 2048)) for _ in range(12)]   # 134 MB of grid each
    for p in plans:
        lib.mnufft_destroy(p)
    assert live() <= 1 << 30
    """)
