"""One-launch measurement of the plain form against its definitions, at the
sides and packings where rows end inside, at and across 32-bit words."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def expected(S, J, refs):
    """unsat, mag, overlap, autocorr, c4 by their definitions (eqs. 1-3, 7);
    S [2][z][y][x], J [d][z][y][x], refs a list of two-replica states or None."""
    axes = (2, 1, 0)
    L = S[0].shape[0]
    q = S[0].astype(np.int64) * S[1]
    unsat = [sum(int((J[d] * s * np.roll(s, -1, ax) < 0).sum()) for d, ax in enumerate(axes)) for s in S]
    auto = [[0 if ref is None else int((S[r].astype(np.int64) * ref[r]).sum()) for ref in refs] for r in (0, 1)]
    c4 = [[int((q * np.roll(q, -rho, ax)).sum()) for rho in range(L // 2 + 1)] for ax in axes]
    return unsat, [int(s.sum(dtype=np.int64)) for s in S], int(q.sum()), auto, c4


@pytest.mark.parametrize("L,rw", [(8, 0), (8, 1), (16, 2), (24, 3), (40, 0), (48, 2), (56, 1), (64, 8), (72, 0),
                                  (88, 0), (96, 3), (120, 0), (128, 16), (200, 0), (256, 0)])
def test_measurement_equals_its_definition(ea_gpu, L, rw):
    """Whole numbers: no tolerance.  Measured twice and after a reset, since
    the counters are never cleared in between."""
    rng = np.random.default_rng(L)
    pm = np.array([-1, 1], dtype=np.int8)
    g = ea_gpu.Sim(L, 0.4, 0.9, seed=L, n_slots=2, words_per_row=rw)
    J = rng.choice(pm, size=3 * L ** 3)
    g.set_bonds(J)
    assert np.array_equal(g.bonds(), J)
    Jd = J.reshape(L, L, L, 3).transpose(3, 0, 1, 2)
    refs = [None, None]

    def put():
        # correlated replicas, so that no count is trivially half
        a = rng.choice(pm, size=L ** 3)
        S = [a, a * np.where(rng.random(L ** 3) < 0.2, -1, 1).astype(np.int8)]
        for r in (0, 1):
            g.set_spins(r, S[r])
            assert np.array_equal(g.spins(r), S[r])
        return [s.reshape(L, L, L) for s in S]

    def check(S):
        o = g.measure()
        unsat, mag, overlap, auto, c4 = expected(S, Jd, refs)
        assert list(o.unsat) == unsat and list(o.mag) == mag and o.overlap == overlap
        assert np.array_equal(o.autocorr, np.array(auto)) and np.array_equal(o.c4, np.array(c4))

    S = put()
    check(S)
    g.snapshot(1)
    refs[1] = S
    check(S)
    S = put()
    part = g.measure(c4=False, autocorr=False)  # leaves the other counters alone
    assert part.overlap == expected(S, Jd, refs)[2]
    check(S)
    g.reset(seed=3)
    g.set_bonds(J)
    refs[1] = None
    check(put())
    g.close()


@pytest.mark.parametrize("L,rw", [(16, 0), (64, 0), (128, 16), (256, 0)])
def test_state_access_between_sweeps_changes_nothing(ea_gpu, L, rw):
    """Reading and writing back the state between sweeps (its conversion uses
    the slab exchange area) leaves the trajectory bit for bit as it is."""
    a, b = (ea_gpu.Sim(L, 0.3, 0.8, seed=7, words_per_row=rw) for _ in range(2))
    for _ in range(3):
        a.sweep(5)
        b.sweep(5)
        for r in (0, 1):
            S = a.spins(r)
            a.set_spins(r, S)
        a.set_bonds(a.bonds())
    b.sweep(4)
    a.sweep(4)
    for r in (0, 1):
        assert np.array_equal(a.spins(r), b.spins(r))
    bad = a.spins(0)
    bad[-1] = 0
    with pytest.raises(ea_gpu.EAError, match="not \\+-1"):
        a.set_spins(0, bad)
    assert np.array_equal(a.spins(0), b.spins(0))
    a.close()
    b.close()
