"""Calls that take device memory on first use, where there is none to be had:
they do without it.  A child process puts a function in front of hipMalloc that
refuses requests above a limit; the library finds it first because it is loaded
first, with its symbols global."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = """
#include <stddef.h>
int (*real_malloc)(void **, size_t);
size_t limit = ~(size_t)0;
int refused;
int hipMalloc(void **p, size_t n)
{
    if (n > limit) { ++refused; *p = 0; return 2; }  /* hipErrorOutOfMemory */
    return real_malloc(p, n);
}
"""

CHILD = """
import ctypes, sys
sys.path.insert(0, {root!r})
import torch  # its runtime is the one the library uses
import numpy as np
shim = ctypes.CDLL({shim!r}, mode=ctypes.RTLD_GLOBAL)
import paper_1411_5512_amd as ea
from paper_1411_5512_amd.workloads import Job
lib = ea.abi.lib()
# the runtime's own hipMalloc: the library's handle resolves in its dependencies
ctypes.c_void_p.in_dll(shim, "real_malloc").value = ctypes.cast(lib.hipMalloc, ctypes.c_void_p).value
limit, refused = ctypes.c_size_t.in_dll(shim, "limit"), ctypes.c_int.in_dll(shim, "refused")
assert ctypes.cast(shim.hipMalloc, ctypes.c_void_p).value != ctypes.cast(lib.hipMalloc, ctypes.c_void_p).value

class short:
    def __init__(self, n): self.n = n
    def __enter__(self): limit.value, refused.value = self.n, 0
    def __exit__(self, *a): limit.value = 2 ** 64 - 1

{body}
print("child ok", flush=True)
"""


def _run(tmp_path, body):
    src, so = tmp_path / "shim.c", tmp_path / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", str(so), str(src)], check=True, timeout=60)
    code = CHILD.format(root=ROOT, shim=str(so), body=body)
    r = subprocess.run([sys.executable, "-u", "-c", code], capture_output=True, text=True, timeout=100, cwd=ROOT)
    assert r.returncode == 0 and "child ok" in r.stdout, (r.returncode, r.stdout[-2000:], r.stderr[-3000:])


def test_shells_without_the_fft_scratch(ea_gpu, tmp_path):
    """The direct route's scratch fits under the limit, the FFT route's does
    not: every side still gives its sums under the automatic route, and sides
    without another form of the FFT refuse only where it is asked for."""
    _run(tmp_path, """
for L in (48, 56, 64, 72):
    s = ea.Sim(L, 0.4, 0.8, seed=L); s.sweep(5)
    want = ea.Sim(L, 0.4, 0.8, seed=L); want.sweep(5)
    with short(400_000):
        got = s.c4_shells()
        assert refused.value == 1, (L, refused.value)
        again = s.c4_shells(100)
    w = want.c4_shells()
    assert np.array_equal(got, w) and np.array_equal(again, w[:100]) and got[0] == L ** 3, L
    assert np.array_equal(s.c4_shells(), w), L  # with memory again
    if L <= 64:
        job = Job(L, 0.4, 0.8, seed=L, n_sweeps=2, meas_t=[2], tw=[])
        b = ea.Batch([job]); b.run()
        with short(400_000):
            got = b.c4_shells(0, 0)
            assert refused.value == 1, L
        c = ea.Batch([job]); c.run()
        assert np.array_equal(got, c.c4_shells(0, 0)), L
    print("shells", L, flush=True)
m, n = (ea.Msc(64, 4, 0.4, 0.8, seed=1) for _ in range(2))
with short(400_000):
    got = m.c4_shells(1)
    assert refused.value == 1
assert np.array_equal(got, n.c4_shells(1))
ea.set_shell_route(ea.SHELLS_FFT)
for L in (64, 72):
    s = ea.Sim(L, 0.4, 0.8, seed=L)
    with short(400_000):
        try:
            s.c4_shells()
            assert L == 72
        except ea.abi.EAError as e:
            assert L == 64 and e.status == ea.abi.EA_ERR_NOMEM, (L, e)
""")


def test_spins_and_couplings_without_a_conversion_buffer(ea_gpu, tmp_path):
    """A packing too fine for the slab path has no exchange area to convert
    in; where there is no room for a buffer either, the arrays still pass."""
    _run(tmp_path, """
L, rw = 96, 12
a = ea.Sim(L, 0.4, 0.8, seed=3, words_per_row=rw); a.sweep(3)
ref = ea.Sim(L, 0.4, 0.8, seed=3); ref.sweep(3)
rng = np.random.default_rng(1)
spins = rng.choice(np.array([-1, 1], dtype=np.int8), size=L ** 3)
bonds = rng.choice(np.array([-1, 1], dtype=np.int8), size=3 * L ** 3)
with short(400_000):
    assert all(np.array_equal(a.spins(r), ref.spins(r)) for r in (0, 1)) and refused.value == 2
    assert np.array_equal(a.bonds().ravel(), ref.bonds().ravel())
    a.set_spins(1, spins); a.set_bonds(bonds)
    assert refused.value == 5, refused.value
ref.set_spins(1, spins); ref.set_bonds(bonds)
assert np.array_equal(a.spins(1), spins) and np.array_equal(a.bonds().ravel(), bonds)
a.sweep(2); ref.sweep(2)
assert all(np.array_equal(a.spins(r), ref.spins(r)) for r in (0, 1))
""")


def test_few_shells_take_no_scratch_array(ea_gpu, tmp_path):
    """Where the direct count of a few shells is the faster call, the automatic
    route makes it and asks for no FFT scratch; past the line it is the FFT."""
    _run(tmp_path, """
for L, few in ((48, 220), (56, 101), (72, 28), (80, 17), (88, 10)):
    want = ea.Sim(L, 0.4, 0.8, seed=L); want.sweep(5)
    w = want.c4_shells()
    for n, asked in ((1, 0), (few, 0), (few + 1, 1)):
        s = ea.Sim(L, 0.4, 0.8, seed=L); s.sweep(5)
        with short(600_000):
            got = s.c4_shells(n)
            assert refused.value == asked, (L, n, refused.value)
        assert np.array_equal(got, w[:n]), (L, n)
s = ea.Sim(64, 0.4, 0.8, seed=64)
with short(600_000):
    s.c4_shells(1)
    assert refused.value == 1
""")
