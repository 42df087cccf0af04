"""GPU test of the prey's move at every lane-group width: two robots on a diagonal
through the prey, the nearer one deciding, leave two candidates whose scores are
equal but for rounding, so that the choice shows the order in which each kernel
rounds them. The state after a step is the same, bit for bit, at any width."""
import numpy as np
import pytest

from tests.gpu_util import banner, ctx_and_lib, host

pytestmark = pytest.mark.gpu


def test_prey_choice_does_not_depend_on_the_lane_group():
    import torch

    R, ctx = ctx_and_lib()
    E, n = 512, 2
    p = R.params(seed=3, scenario=R.RS_SCN_PREDATOR_PREY, controller=R.RS_CTRL_WAYPOINT)
    d = np.random.default_rng(2).uniform(0.3, 0.8, E).astype(np.float32)
    pos = np.stack([d, -d * np.float32(1.0001)], axis=1)
    got = {}
    for lanes in (2, 4, 8, 16):
        banner(f"prey widths lanes={lanes}")
        s = R.RsSchedule()
        s.lanes_per_env[n] = lanes
        plan = R.Plan(ctx, np.full(E, n, np.int32), s)
        b = R.Batch.empty(E, 0, total_robots=plan.total_robots)  # the prey at (0, 0)
        for f in (b.x, b.y):
            f.copy_(torch.from_numpy(pos.ravel()))
        R.env_run(ctx, p, plan, b, 1)
        torch.cuda.synchronize()
        got[lanes] = {f: host(getattr(b, f)) for f in ("x", "y", "theta", "goal_x", "goal_y")}
        plan.close()
    moved = got[2]["goal_x"].reshape(E, n)[:, 0]
    assert (moved > 0).any() and (moved < 0).any()  # both candidates of the pair are taken
    for lanes in (4, 8, 16):
        for f in got[2]:
            np.testing.assert_array_equal(got[lanes][f], got[2][f], err_msg=f"{f} lanes={lanes}")
