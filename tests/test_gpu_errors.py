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
