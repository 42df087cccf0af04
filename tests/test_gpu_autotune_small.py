"""GPU test of the autotuner on a batch that leaves SIMDs idle: envs per wavefront
that it did not measure as a candidate are marked as automatic in the schedule it
returns and in the one it stores, so that a later, larger batch does not inherit
what only suits the small one."""
import pytest

from tests.gpu_util import banner, ctx_and_lib

pytestmark = pytest.mark.gpu


def test_unmeasured_envs_per_wave_stay_automatic():
    R, ctx = ctx_and_lib()
    banner("autotune on a small batch")
    s = R.autotune(ctx, R.params(), [2, 3, 6], envs=200, steps=20, tol=1e-4)
    stored = R.get_schedule(ctx)
    assert bytes(stored) == bytes(s)
    for n in (2, 3, 6):
        full = 64 // s.lanes_per_env[n]
        candidates = {full // d for d in (1, 2, 4, 8) if full // d >= 1}
        marked = (s.envs_per_wave[0] >> n) & 1
        assert marked or s.envs_per_wave[n] in candidates, (n, s.envs_per_wave[n])
    R.set_schedule(ctx, s)  # accepted as it was returned
