"""Measurements taken inside the batched sweep kernel, where the last
workgroup of a job computes the pair observables over its own lattice in LDS
and loads the lattice again."""
import numpy as np
import pytest

from paper_1411_5512_amd.workloads import Job

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,split", [(L, 1) for L in range(8, 65, 8)] + [(L, 2) for L in (48, 56, 64)])
def test_batch_measurement_equals_plain(ea_gpu, L, split):
    """Whole numbers and spins: no tolerance.  Consecutive measurements and
    sweeps between them, so that a lattice not put back shows."""
    times, tw = [0, 1, 2, 7, 12], [1, 5]
    jobs = [Job(L, 0.4, 0.9, seed=L + s, n_sweeps=15, meas_t=times, tw=tw) for s in range(3)]
    b = ea_gpu.Batch(jobs, split=split)
    b.run()
    for i, j in enumerate(jobs):
        assert b.parts(i) == split
        g = ea_gpu.Sim(L, j.p, j.T, seed=j.seed, n_slots=2)
        for t in range(16):
            if t in tw:
                g.snapshot(tw.index(t))
            if t in times:
                got, want = b.result(i, times.index(t)), g.measure()
                assert list(got.unsat) == list(want.unsat) and list(got.mag) == list(want.mag)
                assert got.overlap == want.overlap and np.array_equal(got.c4, want.c4)
                taken = [k for k, w in enumerate(tw) if w <= t]
                assert all(np.array_equal(np.array(got.autocorr)[:, k], np.array(want.autocorr)[:, k]) for k in taken)
            if t < 15:
                g.sweep(1)
        assert all(np.array_equal(b.spins(i, r), g.spins(r)) for r in (0, 1))
        g.close()
    b.close()


@pytest.mark.parametrize("L", [16, 24, 32, 48])
def test_every_packing_measures_the_same(ea_gpu, L):
    """The tuner compares all counters of every configuration with the
    default's."""
    tried = ea_gpu.tune(L, force=True)["tried"]
    assert len({c["words_per_row"] for c in tried}) > 1 and all(c["parity_ok"] for c in tried)
