"""Transfers through the pinned buffer by few threads and by many, once it is
there: made by a transfer of 32 MiB or more, beside steps still queued, for one
of several solves, or after 32 MiB have gone through the runtime.  No arithmetic
is involved, so states come back bit for bit; the moments of one state are the
same bits each time they are read."""
import threading

import numpy as np
import pytest

from paper_1010_4135_amd import inputs

pytestmark = pytest.mark.gpu

# states of just over 4 MiB, ends inside a chunk, just below and above 32 MiB
GRIDS = [(34, 33, 32), (65, 33, 31), (64, 64, 64), (97, 67, 43), (97, 67, 61)]


def _round_trip(c, seed):
    from paper_1010_4135_amd import lbm3d
    with lbm3d.Solver(c.params) as s:
        s.init(*c.fields)
        m = s.moments()
        f = s.get_f()
        g = (f * np.random.default_rng(seed).uniform(0.9, 1.1, f.shape)).astype(f.dtype)
        s.set_f(g)
        return m, f, g, s.get_f()


@pytest.fixture
def buffer():
    """A solve that keeps the buffer that its own large transfers made."""
    from paper_1010_4135_amd import lbm3d
    c = inputs.smooth_periodic(3, grid=(96, 96, 96), precision=inputs.FP64)
    with lbm3d.Solver(c.params) as s:
        s.init(*c.fields)
        s.get_f()
        yield


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
def test_with_the_buffer_there(grid, buffer):
    c = inputs.smooth_periodic(43, grid=grid, precision=inputs.FP64)
    _, f, put, got = _round_trip(c, 1)
    _, f2, put2, got2 = _round_trip(c, 1)
    assert np.array_equal(put, got) and np.array_equal(f, f2) and np.array_equal(got, got2)


def test_read_back_until_the_buffer_is_made():
    from paper_1010_4135_amd import lbm3d
    c = inputs.smooth_periodic(43, grid=(64, 64, 64), precision=inputs.FP64)
    with lbm3d.Solver(c.params) as s:
        s.init(*c.fields)
        first, state = s.moments(), s.get_f()
        for k in range(16):
            assert all(np.array_equal(a, b) for a, b in zip(first, s.moments())), k
        assert np.array_equal(state, s.get_f())


def test_made_beside_queued_steps():
    """Read back with 300 steps queued and with none: the same bits."""
    from paper_1010_4135_amd import lbm3d
    c = inputs.smooth_periodic(43, grid=(64, 64, 64), precision=inputs.FP32)
    out = []
    for wait in (False, True):
        with lbm3d.Solver(c.params) as s:
            s.init(*c.fields)
            s.step(300)
            if wait:
                s.sync()
            m = s.moments()
            s.step(300)
            if wait:
                s.sync()
            out.append((m, s.get_f(), s.moments(), s.status()))
    for a, b in zip(out[0][0] + out[0][2], out[1][0] + out[1][2]):
        assert np.array_equal(a, b)
    assert np.array_equal(out[0][1], out[1][1]) and out[0][3] == out[1][3]


def test_threads_copy_at_once(buffer):
    cases = [inputs.smooth_periodic(43, grid=(64, 64 + 16 * k, 64), precision=inputs.FP64) for k in range(4)]
    out = [None] * len(cases)

    def work(k):
        out[k] = _round_trip(cases[k], k)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(cases))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k, c in enumerate(cases):
        m, f, put, got = out[k]
        assert np.array_equal(put, got)
        m2, f2, _, _ = _round_trip(c, k)
        assert np.array_equal(f, f2) and all(np.array_equal(a, b) for a, b in zip(m, m2))


def test_with_another_device_current():
    """Fields of a solve on device 0 in and out while the caller's thread has
    device 1 current, which it keeps."""
    import ctypes

    from paper_1010_4135_amd import lbm3d
    if lbm3d.lbm3d_device_count() < 2:
        pytest.skip("needs two devices")
    hip = ctypes.CDLL("libamdhip64.so")
    now = ctypes.c_int()
    c = inputs.smooth_periodic(43, grid=(96, 96, 96), precision=inputs.FP64)
    with lbm3d.Solver(c.params) as s:
        s.init(*c.fields)
        want = s.moments()
        try:
            assert hip.hipSetDevice(1) == 0
            s.init(*c.fields)
            got = s.moments()
            assert hip.hipGetDevice(ctypes.byref(now)) == 0 and now.value == 1
        finally:
            hip.hipSetDevice(0)
        assert all(np.array_equal(a, b) for a, b in zip(want, got))
