"""The batched tuner times sweeps, long enough to tell configurations apart, and
leaves the default (the only one that can split) for a clear gain alone."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [24, 32, 48, 64])
def test_choice_beats_the_default_clearly(ea_gpu, L):
    r = ea_gpu.tune(L, force=True)
    default, chosen = r["tried"][0], r["chosen"]
    # 128 workgroups of L = 24 .. 64 do 2 x 96 .. 1024 half-steps of 9.3 .. 1.1 us in the timed span
    assert default["ms"] > 1.65
    same = all(chosen[k] == default[k] for k in ("words_per_row", "threads", "select"))
    assert same or chosen["ms"] < 0.98 * default["ms"]
    if L == 64:
        assert chosen["threads"] == 1024
