"""GPU test of the fused rollout's split wavefronts (few envs per wavefront, for
small batches): every output and the final state equal, bit for bit, those of
the full-wavefront kernel, which a call with qp_stats selects, at every robot
count, with partial last wavefronts, a single env and resets inside the window."""
import numpy as np
import pytest

from paper_2505_06771_amd import synth
from tests.gpu_util import banner, ctx_and_lib, host

pytestmark = pytest.mark.gpu


def _run(R, ctx, p, n, E, H, policy, stats):
    import torch

    D = 2 * n + 4
    b = R.Batch.empty(E, n, env_id_base=3)
    R.env_reset(ctx, p, b)
    b.step += torch.arange(E, dtype=torch.int32, device="cuda") % 7  # resets spread out
    out = {"obs": torch.empty(H * E * n * D, device="cuda"),
           "actions": torch.empty(H * E * n, dtype=torch.uint8, device="cuda"),
           "reward": torch.empty(H * E, device="cuda"),
           "done": torch.empty(H * E, dtype=torch.uint8, device="cuda")}
    qs = torch.zeros(E * R.QPS_COUNT, dtype=torch.int32, device="cuda") if stats else None
    R.rollout(ctx, p, b, policy, H, 11, out["obs"], out["actions"], out["reward"], out["done"],
              qp_stats=qs)
    torch.cuda.synchronize()
    res = {k: host(v) for k, v in out.items()}
    for k in ("x", "y", "theta", "goal_x", "goal_y", "step", "episode"):
        res[k] = host(getattr(b, k))
    return res


@pytest.mark.parametrize("prey", [False, True])
@pytest.mark.parametrize("n", range(2, 15))
def test_split_wavefronts_match_full_ones(n, prey):
    import torch

    R, ctx = ctx_and_lib()
    kw = dict(scenario=R.RS_SCN_PREDATOR_PREY, controller=R.RS_CTRL_WAYPOINT) if prey else {}
    p = R.params(seed=5, max_steps=15, action_noise=0.02 if n % 2 else 0.0, **kw)
    w = synth.policy_weights(n, 2 * n + 4, bias_scale=0.1)
    bf = lambda a: torch.from_numpy(a).to(torch.bfloat16).cuda().contiguous()
    fl = lambda a: torch.from_numpy(a).float().cuda().contiguous()
    pol = R.Policy(bf(w["w1"]), fl(w["b1"]), bf(w["w2"]), fl(w["b2"]), bf(w["w3"]), fl(w["b3"]))
    lanes = 2 if n == 2 else 4 if n <= 4 else 8 if n <= 8 else 16
    tile = max(1, 16 // lanes)
    # one env, several, then several per wavefront with a partial last one: one
    # MLP tile, and two
    for E in (1, 7, 1024 * max(tile // 2, 1) + 3, 1024 * tile + 3):
        banner(f"split rollout n={n} E={E} prey={prey}")
        got = _run(R, ctx, p, n, E, 20, pol, False)
        ref = _run(R, ctx, p, n, E, 20, pol, True)
        for k in ref:
            np.testing.assert_array_equal(got[k], ref[k], err_msg=f"{k} n={n} E={E}")
