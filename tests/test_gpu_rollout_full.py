"""GPU test of the fused rollout's full-wavefront kernels (64 / G envs each), which
launches past the split limit take: at every robot count, both scenarios and all
sampling controllers, every output and the final state equal, bit for bit, those
of the kernel that also counts the certificate's stages (full wavefronts too) and,
for the first and the last envs, those of the split kernel, which small batches
take and which the oracle tests cover."""
import numpy as np
import pytest

from paper_2505_06771_amd import synth
from tests.gpu_util import banner, ctx_and_lib, host

pytestmark = pytest.mark.gpu

STATE = ("x", "y", "theta", "goal_x", "goal_y", "step", "episode")
H = 12


def _run(R, ctx, p, n, first, E, policy, stats=False):
    """Envs first .. first + E of a batch whose resets are spread over the window,
    each output and state field as [E, ...]."""
    import torch

    D = 2 * n + 4
    b = R.Batch.empty(E, n, env_id_base=first)
    R.env_reset(ctx, p, b)
    b.step += (first + torch.arange(E, dtype=torch.int32, device="cuda")) % 7
    obs = torch.empty((H, E, n * D), device="cuda")
    act = torch.empty((H, E, n), dtype=torch.uint8, device="cuda")
    rew = torch.empty((H, E), device="cuda")
    done = torch.empty((H, E), dtype=torch.uint8, device="cuda")
    qs = torch.zeros((E, R.QPS_COUNT), dtype=torch.int32, device="cuda") if stats else None
    R.rollout(ctx, p, b, policy, H, 11, obs, act, rew, done, qp_stats=qs)
    torch.cuda.synchronize()
    res = {k: host(v).swapaxes(0, 1) for k, v in
           (("obs", obs), ("actions", act), ("reward", rew), ("done", done))}
    res.update({k: host(getattr(b, k)).reshape(E, -1) for k in STATE})
    return res


@pytest.mark.parametrize("kind", ["discrete", "waypoint", "pose", "prey"])
@pytest.mark.parametrize("n", range(2, 15))
def test_full_wavefronts_match_stats_and_split_kernels(n, kind):
    import torch

    R, ctx = ctx_and_lib()
    ctrl = {"discrete": R.RS_CTRL_DISCRETE, "pose": R.RS_CTRL_POSE}.get(kind, R.RS_CTRL_WAYPOINT)
    scn = R.RS_SCN_PREDATOR_PREY if kind == "prey" else R.RS_SCN_NAVIGATION
    p = R.params(seed=5, max_steps=10, action_noise=0.02 if n % 2 else 0.0, controller=ctrl,
                 scenario=scn)
    w = synth.policy_weights(n, 2 * n + 4, bias_scale=0.1)
    bf = lambda a: torch.from_numpy(a).to(torch.bfloat16).cuda().contiguous()
    fl = lambda a: torch.from_numpy(a).float().cuda().contiguous()
    pol = R.Policy(bf(w["w1"]), fl(w["b1"]), bf(w["w2"]), fl(w["b2"]), bf(w["w3"]), fl(w["b3"]))
    lanes = 2 if n == 2 else 4 if n <= 4 else 8 if n <= 8 else 16
    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    E = simds * (32 // lanes) + 3  # just past the split limit, a partial last wavefront
    banner(f"full rollout n={n} {kind} E={E}")
    full = _run(R, ctx, p, n, 0, E, pol)
    ref = _run(R, ctx, p, n, 0, E, pol, stats=True)
    for k in ref:
        np.testing.assert_array_equal(full[k], ref[k], err_msg=f"{k} against the stats kernel")
    for first, count in ((0, 5), (E - 4, 4), (simds, 2 * (64 // lanes) + 1)):
        part = _run(R, ctx, p, n, first, count, pol)
        for k in part:
            np.testing.assert_array_equal(full[k][first:first + count], part[k],
                                          err_msg=f"{k} envs {first}.. against split")
