"""Sweeps in calls of one to four: launches shorter than the slabs' ghost
depth, where a slab's write-back must not meet a neighbour's first load."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,n_sims,plan", [(L, n, None) for L in (8, 16, 24, 32, 40, 64) for n in (1, 3)] +
                         [(24, 1, (4, 2)), (24, 1, (4, 3)), (16, 1, (2, 8)), (32, 1, (8, 4))])
def test_short_calls_equal_one_call(ea_gpu, L, n_sims, plan):
    """Spins: no tolerance."""
    runs = [ea_gpu.Sim(L, 0.4, 0.8, seed=L + s) for s in range(n_sims)]
    whole = [ea_gpu.Sim(L, 0.4, 0.8, seed=L + s) for s in range(n_sims)]
    if plan:
        runs[0].set_slab_plan(*plan)
        assert runs[0].slab_plan == plan
    total = 0
    for k in range(400):
        n = 1 + k % 4
        ea_gpu.sweep_group(runs, n) if n_sims > 1 else runs[0].sweep(n)
        total += n
    for a, b in zip(runs, whole):
        b.sweep(total)
        assert all(np.array_equal(a.spins(r), b.spins(r)) for r in (0, 1))
    for s in runs + whole:
        s.close()
