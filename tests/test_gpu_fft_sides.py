"""Full-vector C4 by FFT at L = 2^k and 3 2^k, and the dense overlap rows of
every packing, against numpy's FFT."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def shells_of(q):
    """Shell sums of the periodic autocorrelation of q."""
    L = q.shape[0]
    f = np.fft.fftn(q.astype(np.float64))
    corr = np.rint(np.fft.ifftn(f * f.conj()).real).astype(np.int64)
    m = np.minimum(np.arange(L), L - np.arange(L)) ** 2
    out = np.zeros(3 * (L // 2) ** 2 + 1, dtype=np.int64)
    np.add.at(out, (m[:, None, None] + m[None, :, None] + m[None, None, :]).ravel(), corr.ravel())
    return out


# rw: the coarsest packing, the finest (words of four sites) and one between
@pytest.mark.parametrize("L,rw", [(L, rw) for L in (8, 16, 24, 32, 40, 48, 56, 64, 72, 96, 128) for rw in (0, L // 8)] +
                         [(48, 2), (80, 2), (128, 4), (192, 0), (256, 0), (256, 8)])
def test_fft_shells(ea_gpu, L, rw):
    """Whole numbers: no tolerance.  The second call is shorter: what the
    first left behind is cleared."""
    rng = np.random.default_rng(L)
    pm = np.array([-1, 1], dtype=np.int8)
    noise = rng.standard_normal((L, L, L))
    q = np.where(noise + np.roll(noise, 1, 0) + np.roll(noise, 1, 2) > 0, 1, -1).astype(np.int8)
    s = ea_gpu.Sim(L, 0.5, 0.8, seed=1, words_per_row=rw)
    a = rng.choice(pm, size=L ** 3)
    s.set_spins(0, a)
    s.set_spins(1, a * q.ravel())
    want = shells_of(q)
    try:
        ea_gpu.set_shell_route(ea_gpu.SHELLS_FFT)
        assert np.array_equal(s.c4_shells(len(want)), want)
        n = (L // 2) ** 2 + 1
        assert np.array_equal(s.c4_shells(n), want[:n])
        if L <= 96:
            ea_gpu.set_shell_route(ea_gpu.SHELLS_DIRECT)
            assert np.array_equal(s.c4_shells(n), want[:n])
    finally:
        ea_gpu.set_shell_route(ea_gpu.SHELLS_AUTO)
    s.close()
