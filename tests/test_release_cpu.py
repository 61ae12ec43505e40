"""When a plan's or batch's memory may go to the next one: the library's host code
with a stand-in for the HIP runtime, which counts the waits."""
import pytest

from tests import host_shim

S1, S2 = 0x51000, 0x52000


@pytest.mark.parametrize("call", [
    "lib.mnufft_execute(h, P[3], P[4])",
    "lib.mnufft_execute_adjoint(h, P[3], P[4])",
    "lib.mnufft_execute_sorted(h, P[3], P[4])",
    "lib.mnufft_spread(h, P[3], P[4])",
    "lib.mnufft_interp(h, P[3], P[4])",
    "lib.mnufft_interp_grad(h, P[3], P[4], P[5], P[6], None)",
    "lib.mnufft_get_sort(h, P[3], P[4])",
    "lib.mnufft_get_subproblems(h, P[3], P[4])",
    "setpts(h, 1000, 2)",
])
@pytest.mark.parametrize("how", ["destroy", "grow"])
def test_captured_plan_waits_for_the_device(tmp_path, call, how):
    """A captured call may be replayed on any stream: the plan's own stream being
    idle does not free its memory."""
    host_shim.run(tmp_path, f"""
    for capture in (False, True):
        h = plan(1, (64, 64), stream={S1})
        assert setpts(h, 1000, 2) == 0
        fake.fake_capture({S1} if capture else None)
        assert {call} == 0
        fake.fake_capture(None)
        fake.fake_clear()
        if "{how}" == "grow":
            assert setpts(h, 5000, 2) == 0
            assert (count(DEVICE_SYNC) > 0) == capture
        assert lib.mnufft_destroy(h) == 0
        assert (count(DEVICE_SYNC) > 0) == capture
    """)


def test_captured_type3_sub_plans(tmp_path):
    """The plans inside a type 3 plan are made anew when its grid changes."""
    host_shim.run(tmp_path, f"""
    for capture in (False, True):
        h = plan(3, (1, 1), stream={S1})
        assert lib.mnufft_setpts3(h, 100, P[0], P[1], None, 50, P[2], P[3], None) == 0
        fake.fake_capture({S1} if capture else None)
        assert lib.mnufft_execute(h, P[3], P[4]) == 0
        fake.fake_capture(None)
        fake.fake_clear()
        fake.fake_bounds(ctypes.c_double(30.0))     # a larger space-bandwidth product
        assert lib.mnufft_setpts3(h, 100, P[0], P[1], None, 50, P[2], P[3], None) == 0
        fake.fake_bounds(ctypes.c_double(0.0))
        assert (count(DEVICE_SYNC) > 0) == capture
        lib.mnufft_destroy(h)
    """)


@pytest.mark.parametrize("type_", [1, 2])
def test_captured_batch_waits_for_the_device(tmp_path, type_):
    host_shim.run(tmp_path, f"""
    for what in ("none", "setpts", "execute"):
        h = batch({type_}, [(64, 60), (32, 40)], [1000, 500], stream={S1})
        fake.fake_capture({S1} if what == "setpts" else None)
        assert lib.mnufft_batch_setpts(h, P[0], P[1], None) == 0
        fake.fake_capture({S1} if what == "execute" else None)
        assert lib.mnufft_batch_execute(h, P[3], P[4]) == 0
        fake.fake_capture(None)
        fake.fake_clear()
        assert lib.mnufft_batch_destroy(h) == 0
        assert (count(DEVICE_SYNC) > 0) == (what != "none"), what
    """)


def test_wait_on_the_plans_device(tmp_path):
    """A plan made on the current device (device -1) waits for that device when
    another is current at its end."""
    host_shim.run(tmp_path, f"""
    for stream in (None, {S1}):
        lib.mnufft_destroy(plan(1, (64, 64)))       # (its memory stays in the pool)
        fake.hipSetDevice(1)
        h = plan(1, (64, 64), stream=stream)
        b = batch(1, [(64, 60)], [1000], stream=stream)
        fake.hipSetDevice(0)
        lib.mnufft_destroy(h)
        assert count(SYNC_DEV) == 1
        lib.mnufft_batch_destroy(b)
        assert count(SYNC_DEV) == 1
        d = ci(-1)
        fake.hipGetDevice(ctypes.byref(d))
        assert d.value == 0
    """)


def test_memory_is_returned_when_a_wait_fails(tmp_path):
    """Memory that may still be in use is freed, which waits for its users, and is
    not handed to the next plan."""
    host_shim.run(tmp_path, f"""
    h = plan(1, (64, 64), stream={S1})
    assert setpts(h, 1000, 2) == 0
    fake.fake_fail_waits(1)
    fake.fake_clear()
    assert lib.mnufft_destroy(h) == -3
    fake.fake_fail_waits(0)
    assert live() == 0
    """)


def test_per_thread_stream(tmp_path):
    """The per-thread stream of the thread that destroys need not be the one used."""
    host_shim.run(tmp_path, """
    h = plan(1, (64, 64), stream=2)                 # hipStreamPerThread
    assert setpts(h, 1000, 2) == 0
    fake.fake_clear()
    lib.mnufft_destroy(h)
    assert count(DEVICE_SYNC) > 0
    """)


def test_stream_destroyed_before_the_plan_moves(tmp_path):
    """Moving a plan does not touch the stream that it leaves."""
    host_shim.run(tmp_path, f"""
    h = plan(1, (64, 64), stream={S1})
    assert setpts(h, 1000, 2) == 0
    fake.fake_stream_gone({S1})
    assert lib.mnufft_set_stream(h, {S2}) == 0
    assert lib.mnufft_execute(h, P[3], P[4]) == 0
    assert count(OVERRUN) == 0
    lib.mnufft_destroy(h)
    """)
