"""GPU test of the env split over wavefronts in env_step, env_steps and
barrier_certificate: a batch large enough for full or part-filled wavefronts
gives, bit for bit, what the same envs give in small batches (one env per
wavefront, the other lanes running along), partial last wavefronts included."""
import numpy as np
import pytest

from paper_2505_06771_amd import synth
from tests.gpu_util import banner, batch_from_states, ctx_and_lib, dev, host

pytestmark = pytest.mark.gpu

FIELDS = ("x", "y", "theta", "goal_x", "goal_y", "step", "episode")


def _states(seed, E, n):
    """E envs from a few hundred distinct ones (drawing them is slow)."""
    k = 300
    st = synth.random_states(seed, k, n)
    crowd = synth.stressed_states(seed + 1, k, n, "mixed")
    pick = np.arange(E)
    return {f: np.where((pick % 8 == 7)[:, None], crowd[f][pick % k], st[f][pick % k]) for f in st}


@pytest.mark.parametrize("kind", ["f32", "f64"])
@pytest.mark.parametrize("n,E", [(2, 300), (2, 9000), (3, 4097), (7, 2051), (16, 1030), (16, 2051)])
def test_large_batch_equals_small_ones(n, E, kind):
    import torch

    R, ctx = ctx_and_lib()
    tdt = torch.float32 if kind == "f32" else torch.float64
    p = R.params(seed=4, dtype=R.RS_F64 if kind == "f64" else R.RS_F32, max_steps=3)
    st = _states(17 + n, E, n)
    banner(f"wave split n={n} E={E} {kind}")

    def run(lo, hi):
        e = hi - lo
        part = {f: v[lo:hi] for f, v in st.items()}
        b = batch_from_states(R, part, n, tdt, env_id_base=lo)
        obs = torch.empty(e * n * (2 * n + 4), dtype=tdt, device="cuda")
        rew = torch.empty(4 * e, dtype=tdt, device="cuda")
        done = torch.empty(4 * e, dtype=torch.uint8, device="cuda")
        R.env_step(ctx, p, b, t_global=9, obs=obs, reward=rew[:e], done=done[:e])
        R.env_steps(ctx, p, b, 3, t_global0=10, reward=rew[e:], done=done[e:])
        ux, uy = (torch.empty(e * n, dtype=tdt, device="cuda") for _ in range(2))
        lam = torch.empty(e * n * (n - 1) // 2, dtype=tdt, device="cuda")
        cmd = [dev(v.reshape(-1), tdt) for v in synth.nominal_commands(5, (E, n))]
        px, py = (dev(part[f].reshape(-1), tdt) for f in ("x", "y"))
        R.barrier_certificate(ctx, p, e, n, px, py, cmd[0][lo * n:hi * n].contiguous(),
                              cmd[1][lo * n:hi * n].contiguous(), ux, uy, lam=lam)
        torch.cuda.synchronize()
        out = {"obs": host(obs).reshape(e, -1), "reward": host(rew).reshape(4, e).T,
               "done": host(done).reshape(4, e).T, "ux": host(ux).reshape(e, n),
               "uy": host(uy).reshape(e, n), "lam": host(lam).reshape(e, -1)}
        for f in FIELDS:
            out[f] = host(getattr(b, f)).reshape(e, -1)
        return out

    whole = run(0, E)
    for lo, hi in ((0, 1), (1, 70), (E - 131, E)):
        part = run(lo, hi)
        for k in whole:
            np.testing.assert_array_equal(whole[k][lo:hi], part[k], err_msg=f"{k} envs {lo}..{hi}")
