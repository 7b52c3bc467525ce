"""The batched update at the launch shapes whose waves drift between
half-steps or meet at a barrier, with rows packed every way the kernel takes."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [8, 16, 32, 48, 56])
def test_every_launch_shape_gives_the_same_bits(ea_gpu, L):
    """Every packing, thread count (waves that share a plane, that own whole
    planes, and that straddle two) and select variant of one lattice size
    reproduces the default configuration's measurements and spins exactly
    (whole numbers: no tolerance)."""
    out = ea_gpu.tune(L, force=True)
    assert len(out["tried"]) > 1
    assert all(c["parity_ok"] for c in out["tried"]), out["tried"]
