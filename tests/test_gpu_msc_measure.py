"""Measurements of the multispin batch against their definitions, at the line
lengths, slab counts and word sets where the C4 tiles have remainders."""
import numpy as np
import pytest

from test_gpu_measure import expected

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,samples", [(8, 8), (8, 32), (16, 4), (24, 16), (40, 32), (48, 4), (64, 1), (72, 32),
                                       (96, 2), (136, 32), (64, 96)])
def test_measurement_equals_its_definition(ea_gpu, L, samples):
    """Whole numbers: no tolerance.  Twice, with a snapshot of a sample's
    earlier state."""
    rng = np.random.default_rng(L + samples)
    pm = np.array([-1, 1], dtype=np.int8)
    m = ea_gpu.Msc(L, samples, 0.4, 0.9, seed=5, n_slots=1)
    chosen = sorted({0, samples // 2, samples - 1})
    J = {b: m.bonds(b).reshape(L, L, L, 3).transpose(3, 0, 1, 2) for b in chosen}
    refs = {b: None for b in chosen}
    for turn in range(2):
        S = {}
        for b in chosen:
            a = rng.choice(pm, size=L ** 3)
            S[b] = [a, a * np.where(rng.random(L ** 3) < 0.2, -1, 1).astype(np.int8)]
            for r in (0, 1):
                m.set_spins(b, r, S[b][r])
            S[b] = [s.reshape(L, L, L) for s in S[b]]
        obs = m.measure()
        assert len(obs) == samples
        for b in chosen:
            unsat, mag, overlap, auto, c4 = expected(S[b], J[b], [refs[b]])
            o = obs[b]
            assert list(o.unsat) == unsat and list(o.mag) == mag and o.overlap == overlap
            assert np.array_equal(o.autocorr, np.array(auto)) and np.array_equal(o.c4, np.array(c4))
        m.snapshot(0)
        refs = S
    m.close()
