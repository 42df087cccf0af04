"""GPU test of the default spreading of env_run's envs over wavefronts: mixes
whose 16-lane teams take one env per wavefront, several, or full ones (at one
and two wavefronts per SIMD) give, bit for bit, what full wavefronts give, and
so does env_run_noalloc, whose launch has to hold every tile made."""
import numpy as np
import pytest

from tests.gpu_util import banner, ctx_and_lib, host

pytestmark = pytest.mark.gpu

FIELDS = ("x", "y", "theta", "goal_x", "goal_y", "step", "episode")


@pytest.mark.parametrize("mix", [
    {12: 1},
    {16: 1025, 2: 65},             # one env per wavefront, past one wavefront per SIMD
    {9: 2047, 8: 3},
    {16: 2049},                    # two, the last wavefront with one
    {12: 819, 8: 1638, 6: 2458, 4: 2458, 2: 819},
    {16: 8200, 3: 17},             # beyond both limits: full
], ids=str)
def test_spread_equals_full_wavefronts(mix):
    import torch

    R, ctx = ctx_and_lib()
    counts = np.random.default_rng(1).permutation(
        np.concatenate([np.full(e, n, np.int32) for n, e in mix.items()]))
    E, steps = len(counts), 4
    full = R.RsSchedule()
    full.block_threads = 256
    for n in range(2, 17):
        full.envs_per_wave[n] = 64 // (1 << (n - 1).bit_length())
    p = R.params(seed=6, max_steps=4)
    banner(f"run spread {mix}")

    def run(call):
        plan = R.Plan(ctx, counts, full if call == "full" else None)
        b = R.Batch.empty(E, 0, total_robots=plan.total_robots)
        R.env_reset_mixed(ctx, p, plan, b)
        reward = torch.empty((steps, E), device="cuda")
        done = torch.empty((steps, E), dtype=torch.uint8, device="cuda")
        out = {"reward_out": reward, "done_out": done}
        if call == "noalloc":
            R.env_run_noalloc(ctx, p, torch.from_numpy(counts).cuda(), b, steps, 3, **out)
        else:
            R.env_run(ctx, p, plan, b, steps, 3, **out)
        torch.cuda.synchronize()
        got = {f: host(getattr(b, f)) for f in FIELDS}
        got.update(reward=host(reward), done=host(done))
        plan.close()
        return got

    want = run("full")
    for call in ("plan", "noalloc"):
        got = run(call)
        for k in want:
            np.testing.assert_array_equal(got[k], want[k], err_msg=f"{call} {k}")
