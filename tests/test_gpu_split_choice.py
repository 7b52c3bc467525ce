"""Which samples of an uneven batch are split into slabs follows the half-step
times of the sizes, whole and split."""
import pytest

pytestmark = pytest.mark.gpu


# the sweeps are chosen so that the right-hand split shortens the batch by 10%
# or more with the measured times (whole 8.3, 9.3 us at L = 56, 64; slab 4.2, 5.6)
@pytest.mark.parametrize("jobs,parts", [
    ([(64, 2000)], [2]),
    ([(56, 2000)], [2]),
    ([(48, 2000)], [2]),
    ([(64, 2000), (56, 1500)], [2, 2]),
    ([(64, 2000), (56, 1000)], [2, 1]),
    ([(64, 2000), (40, 1000)], [2, 1]),
])
def test_what_splits(ea_gpu, jobs, parts):
    from paper_1411_5512_amd.workloads import Job
    b = ea_gpu.Batch([Job(L, 0.4, 0.8, seed=i, n_sweeps=n, meas_t=[n], tw=[]) for i, (L, n) in enumerate(jobs)])
    assert [b.parts(i) for i in range(len(jobs))] == parts
    b.close()
