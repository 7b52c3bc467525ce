"""Reading a batch's results: in any order, between runs, after a reset, and
at the cost of the rows that are new."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _row(o):
    return np.concatenate([[o.t, o.overlap], o.unsat, o.mag, o.autocorr.ravel(), o.c4.ravel()])


def test_rows_in_any_order_and_between_runs(ea_gpu):
    from paper_1411_5512_amd.workloads import Job
    # enough rows of L = 16 that one copy does not hold them all
    jobs = [Job(L, 0.4, 0.8, seed=i, n_sweeps=n, meas_t=list(range(1, n + 1)), tw=[1])
            for i, (L, n) in enumerate([(16, 900), (8, 5), (24, 40)])]
    whole = ea_gpu.Batch(jobs)
    whole.run()
    want = [[_row(whole.result(j, k)) for k in range(len(job.meas_t))] for j, job in enumerate(jobs)]
    for j in range(3):
        for k in range(len(want[j]) - 1, -1, -1):
            assert np.array_equal(_row(whole.result(j, k)), want[j][k]), (j, k)
    part = ea_gpu.Batch(jobs)
    for again in range(2):
        for t in (1, 3, 7, 8, 400, 900):
            part.run(t)
            for j, job in enumerate(jobs):
                done = min(t, job.n_sweeps)
                for k in {0, done // 2, done - 1}:
                    assert np.array_equal(_row(part.result(j, k)), want[j][k]), (again, t, j, k)
                if done < job.n_sweeps:
                    with pytest.raises(ea_gpu.abi.EAError):
                        part.result(j, done)
        part.reset()
    part.close()
    whole.close()


def test_a_new_row_costs_a_row(ea_gpu):
    """One sweep, one new measurement, read: with 6000 rows in all (960 KB) as
    with 60, within a factor that a copy of them all would pass."""
    from paper_1411_5512_amd.workloads import Job
    took = {}
    for n in (60, 6000):
        b = ea_gpu.Batch([Job(8, 0.4, 0.8, seed=1, n_sweeps=n, meas_t=list(range(1, n + 1)), tw=[])])
        times = []
        for t in range(1, 51):
            b.run(t)
            start = time.perf_counter()
            b.result(0, t - 1)
            times.append(time.perf_counter() - start)
        took[n] = sorted(times)[len(times) // 2]
        b.close()
    print(took)
    assert took[6000] < 1.5 * took[60], took
