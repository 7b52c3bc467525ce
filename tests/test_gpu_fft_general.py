"""Full-vector C4 by FFT at the sides with an odd factor above 3, against the
direct route and numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture
def routes(ea_gpu):
    yield ea_gpu
    ea_gpu.set_shell_route(ea_gpu.SHELLS_AUTO)


def shells_of(q):
    """Shell sums of the periodic autocorrelation of q by numpy's FFT."""
    L = q.shape[0]
    f = np.fft.fftn(q.astype(np.float64))
    corr = np.rint(np.fft.ifftn(f * f.conj()).real).astype(np.int64)
    m = np.minimum(np.arange(L), L - np.arange(L)) ** 2
    shell = (m[:, None, None] + m[None, :, None] + m[None, None, :]).ravel()
    out = np.zeros(3 * (L // 2) ** 2 + 1, dtype=np.int64)
    np.add.at(out, shell, corr.ravel())
    return out


# every factor m of L = m P, each with the P it comes with; the largest side
@pytest.mark.parametrize("L,kind", [(L, "domains") for L in (40, 56, 72, 80, 88, 104, 112, 120, 136, 144, 152, 160, 168,
                                                             184, 200, 216, 224, 232, 240, 248)] +
                         [(L, kind) for L in (40, 136, 248) for kind in ("uniform", "checkerboard")])
def test_general_sides(routes, L, kind):
    """Whole numbers: no tolerance.  A uniform and a checkerboard overlap put
    all of |F|^2 on one wave vector, the hardest case for the rounding."""
    ea = routes
    rng = np.random.default_rng(L)
    z, y, x = np.indices((L, L, L), sparse=True)
    if kind == "uniform":
        q = np.ones((L, L, L), dtype=np.int8)
    elif kind == "checkerboard":
        q = (1 - 2 * ((x + y + z) & 1)).astype(np.int8)
    else:
        noise = rng.standard_normal((L, L, L))
        q = np.where(noise + np.roll(noise, 1, 0) + np.roll(noise, 1, 2) > 0, 1, -1).astype(np.int8)
    s = ea.Sim(L, 0.5, 0.8, seed=1)
    a = rng.choice(np.array([-1, 1], dtype=np.int8), size=L ** 3)
    s.set_spins(0, a)
    s.set_spins(1, a * q.ravel())
    full = 3 * (L // 2) ** 2 + 1
    ea.set_shell_route(ea.SHELLS_FFT)
    got = s.c4_shells(full)
    assert np.array_equal(got, shells_of(q))
    assert np.array_equal(s.c4_shells(), got[: (L // 2) ** 2 + 1])
    if L <= 104:
        ea.set_shell_route(ea.SHELLS_DIRECT)
        assert np.array_equal(s.c4_shells(full), got)
    s.close()


@pytest.mark.parametrize("L", [40, 56])
def test_batched_configurations(routes, L):
    ea = routes
    from paper_1411_5512_amd.workloads import Job
    b = ea.Batch([Job(L, 0.4, 0.8, seed=3, n_sweeps=20, meas_t=[5, 20], tw=[])])
    b.run()
    ea.set_shell_route(ea.SHELLS_DIRECT)
    want = [b.c4_shells(0, k) for k in (0, 1)]
    ea.set_shell_route(ea.SHELLS_FFT)
    assert all(np.array_equal(b.c4_shells(0, k), want[k]) for k in (0, 1))
    b.close()
