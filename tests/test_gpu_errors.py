"""Calls that fail part-way leave nothing behind that a later call would count:
an error that is pending on the thread (here from an allocation of the
caller's own that cannot be had) ends the call it meets, and a retry is right."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _leave_error(ea):
    """A failed hipMalloc, whose error stays pending on this thread."""
    p = ctypes.c_void_p()
    assert ea.abi.lib().hipMalloc(ctypes.byref(p), ctypes.c_size_t(1 << 60)) != 0


def _same(a, b):
    assert a.t == b.t and a.overlap == b.overlap
    for x in ("unsat", "mag", "autocorr", "c4"):
        assert np.array_equal(getattr(a, x), getattr(b, x)), x


@pytest.mark.parametrize("L", [8, 40, 64])
def test_measurement_after_one_that_failed(ea_gpu, L):
    s = ea_gpu.Sim(L, 0.4, 0.8, seed=L, n_slots=1)
    s.snapshot(0)
    s.sweep(7)
    want = s.measure()
    for _ in range(2):
        _leave_error(ea_gpu)
        with pytest.raises(ea_gpu.abi.EAError):
            s.measure()
    _same(s.measure(), want)
    _same(s.measure(), want)
    # a reset that reports the pending error has still started the new sample
    _leave_error(ea_gpu)
    with pytest.raises(ea_gpu.abi.EAError):
        s.reset(seed=L, sample=0)
    s.snapshot(0)
    s.sweep(7)
    _same(s.measure(), want)
    s.close()


def test_allocation_failure_does_not_stay_pending(ea_gpu):
    """A call that reports EA_ERR_NOMEM leaves no error for the next one."""
    s = ea_gpu.Sim(16, 0.4, 0.8, seed=1)
    want = s.measure()
    with pytest.raises(ea_gpu.abi.EAError):
        ea_gpu.Server(hbm_budget=1 << 58)
    _same(s.measure(), want)
    s.sweep(1)
    s.sync()
    s.close()


@pytest.mark.parametrize("L", [8, 16, 40])
def test_couplings_after_a_launch_that_gave_up(ea_gpu, L):
    """A slab launch that gave up leaves the spins undefined, not the couplings.
    The error word is set from here; it lies 192 bytes before the exchange
    area, the last part of the caller's buffer, of 32 bytes per word of a plane
    and slot."""
    s = ea_gpu.Sim(L, 0.4, 0.8, seed=5)
    s.sweep(1)
    s.sync()
    want = s.bonds()
    plane = L * L * s.words_per_row
    aligned = (s._buf.data_ptr() + 255) // 256 * 256 - s._buf.data_ptr()
    end = aligned + s._buf.numel() - 256
    gave_up = False
    for slots in range(1, 9):
        at = end - 32 * plane * slots - 192
        s._buf[at] = 1
        try:
            s.sync()
        except ea_gpu.abi.EAError as e:
            gave_up = e.status == ea_gpu.abi.EA_ERR_DEVICE
            break
    assert gave_up
    for call in (s.measure, lambda: s.spins(0)):
        with pytest.raises(ea_gpu.abi.EAError):
            call()
    assert np.array_equal(s.bonds(), want)
    s.set_bonds(-want)
    assert np.array_equal(s.bonds(), -want)
    # a reset clears the word, and the counters with it
    s.reset(seed=5, sample=0)
    t = ea_gpu.Sim(L, 0.4, 0.8, seed=5)
    s.sweep(4)
    t.sweep(4)
    _same(s.measure(), t.measure())
    assert np.array_equal(s.bonds(), want) and all(np.array_equal(s.spins(r), t.spins(r)) for r in (0, 1))
    s.close()
    t.close()
