"""Launches whose workgroups wait for each other, on several streams at once:
each needs the device (nearly) to itself, so they take turns."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_runs_on_their_own_streams_take_turns(ea_gpu):
    """Runs of L = 128 and 64 swept in short calls, first from one thread
    without waiting, then from a thread each, reach the states they reach
    alone."""
    par = [(128, 1), (64, 2), (128, 3), (96, 4)]
    runs = [ea_gpu.Sim(L, 0.4, 0.8, seed=s) for L, s in par]
    alone = [ea_gpu.Sim(L, 0.4, 0.8, seed=s) for L, s in par]
    for a in alone:
        a.sweep(90)
        a.sync()
    for _ in range(30):
        for r in runs:
            r.sweep(1)

    def work(r):
        for _ in range(20):
            r.sweep(3)
        r.sync()

    threads = [threading.Thread(target=work, args=(r,)) for r in runs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for r, a in zip(runs, alone):
        assert all(np.array_equal(r.spins(k), a.spins(k)) for k in (0, 1))
    for s in runs + alone:
        s.close()
