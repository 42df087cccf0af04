"""GPU tests of env_step, env_steps and barrier_certificate with full wavefronts
(64 / G envs each, the last one partial), whose lane groups are in different
stages of the certificate at the same time: commands against the FP64 oracle, and
bit for bit what the same envs give in small batches (one env per wavefront)."""
import numpy as np
import pytest

from paper_2505_06771_amd import synth
from tests.gpu_util import banner, ctx_and_lib, dev, host
from tests.test_gpu_qp_general import _packs as dense_packs
from tests.test_gpu_qp_thin import _packs as thin_packs
from tests.test_gpu_wave_split import test_large_batch_equals_small_ones as _large_equals_small

pytestmark = pytest.mark.gpu


def _full_batch(n, kind):
    """Envs that fill every wavefront of the launch limit, and three more."""
    import torch

    cus = torch.cuda.get_device_properties(0).multi_processor_count
    lanes = 2 if n == 2 else 4 if n <= 4 else 8 if n <= 8 else 16
    waves = cus * (8 if lanes > 8 and kind == "f32" else 4)
    return waves * (64 // lanes) + 3


def _certificates(R, ctx, p, n, arrs, tdt):
    import torch

    E = arrs[0].shape[0]
    ux, uy = (torch.zeros(E * n, dtype=tdt, device="cuda") for _ in range(2))
    lam = torch.full((E * (n * (n - 1) // 2),), -1.0, dtype=tdt, device="cuda")
    status = torch.full((E,), 255, dtype=torch.uint8, device="cuda")
    qs = torch.zeros((E, R.QPS_COUNT), dtype=torch.int32, device="cuda")
    R.barrier_certificate(ctx, p, E, n, *(dev(a.ravel(), tdt) for a in arrs), ux, uy, lam=lam,
                          infeasible=status, qp_stats=qs)
    torch.cuda.synchronize()
    return {"ux": host(ux).reshape(E, n), "uy": host(uy).reshape(E, n),
            "lam": host(lam).reshape(E, -1), "status": host(status), "stages": host(qs)}


@pytest.mark.parametrize("kind", ["f32", "f64"])
@pytest.mark.parametrize("n", [4, 5, 8, 9, 16])
def test_dense_packs_among_easy_envs(orc, n, kind):
    import torch

    R, ctx = ctx_and_lib()
    tdt, ndt = (torch.float32, np.float32) if kind == "f32" else (torch.float64, np.float64)
    E, K = _full_batch(n, kind), 50
    banner(f"full wavefronts n={n} {kind} E={E}")
    rng = np.random.default_rng(n)
    easy = synth.random_states(70 + n, 200, n)
    cmd = synth.nominal_commands(71 + n, (200, n))
    pool = [np.concatenate([d, e]).astype(ndt) for d, e in
            zip(dense_packs(72 + n, K, n), (easy["x"], easy["y"], *cmd))]
    # a third of the envs dense, in no order; every distinct one at least once
    pick = np.where(rng.random(E) < 0.33, rng.integers(0, K, E), rng.integers(K, K + 200, E))
    pick[rng.permutation(E)[:K + 200]] = np.arange(K + 200)
    p = R.params(dtype=R.RS_F64 if kind == "f64" else R.RS_F32)
    got = _certificates(R, ctx, p, n, [a[pick] for a in pool], tdt)
    alone = _certificates(R, ctx, p, n, pool, tdt)
    for k in got:
        np.testing.assert_array_equal(got[k], alone[k][pick], err_msg=k)
    if n >= 8:
        assert got["stages"][:, R.QPS_GENERAL].sum() > E // 10
    assert got["stages"][:, R.QPS_BOX:R.QPS_TWO_ROWS].sum() > E // 10
    tol = 1e-4 if kind == "f32" else 1e-9
    po = orc.Params()
    for e in range(K + 50):
        at = np.flatnonzero(pick == e)
        ref = orc.barrier_certificate(po, *[a[e].astype(np.float64) for a in pool])
        assert (got["status"][at] == (1 if ref[3] else 0)).all()
        assert max(np.abs(got["ux"][at] - ref[0]).max(), np.abs(got["uy"][at] - ref[1]).max()) <= tol


@pytest.mark.parametrize("kind", ["f32", "f64"])
def test_second_attempts_beside_other_groups(kind):
    """Rows left a sliver by the bounds (solved at the second attempt), packs for
    the general solver and idle envs in the same wavefronts."""
    import torch

    R, ctx = ctx_and_lib()
    tdt, ndt = (torch.float32, np.float32) if kind == "f32" else (torch.float64, np.float64)
    n, K, angle = 8, 48, 2e-5 if kind == "f32" else 1e-10
    E = _full_batch(n, kind)
    banner(f"second attempts {kind} E={E}")
    kw, thin, _ = thin_packs(3, K, angle, 0.14 * angle * np.sqrt(2), False)
    pool = [np.concatenate([a, a, a]).astype(ndt) for a in thin]
    pool[2][K:2 * K, :2] *= -1  # the pair drives together: no thin row
    pool[2][2 * K:], pool[3][2 * K:] = 0, 0
    pool[2][2 * K:, 0], pool[2][2 * K:, 1] = 0.1, -0.1
    pool[1][2 * K:, 0] += ndt(0.5)  # apart
    pick = np.random.default_rng(4).integers(0, 3 * K, E)
    p = R.params(dtype=R.RS_F64 if kind == "f64" else R.RS_F32, **kw)
    got = _certificates(R, ctx, p, n, [a[pick] for a in pool], tdt)
    alone = _certificates(R, ctx, p, n, pool, tdt)
    for k in got:
        np.testing.assert_array_equal(got[k], alone[k][pick], err_msg=k)
    assert (alone["status"][:K] == 0).all() and (alone["stages"][:K, R.QPS_GENERAL] == 1).all()


@pytest.mark.parametrize("kind", ["f32", "f64"])
@pytest.mark.parametrize("n", [4, 5, 8, 9, 16])
def test_steps_of_a_full_launch_equal_small_ones(n, kind):
    _large_equals_small(n, _full_batch(n, kind), kind)
