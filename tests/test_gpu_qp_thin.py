"""GPU test of the certificate with a pair row that the active bounds leave only
a sliver of: two overlapping robots side by side in a narrow arena, whose walls
hold both along their line of centres, so that the row is met by moving across
it (an angle of 2e-6 to 1e-4 rad in FP32, 2e-11 to 1e-9 in FP64), beside a dense
pack that sends the solve to the general solver. Status and commands against the
FP64 oracle."""
import numpy as np
import pytest

from tests.gpu_util import banner, ctx_and_lib, dev, host

pytestmark = pytest.mark.gpu

D, RS, GAIN, X_MAX = 0.1, 0.17, 100.0, 0.285


def _packs(seed, E, angle, v, tiny):
    """Parameters and E envs of 8 robots: the pair at (+-D/2, 0), its centres
    `angle` off the axis, its row violated by v (normalised) at the walls'
    limits, and six robots on a jittered lattice commanded together."""
    rng = np.random.default_rng(seed)
    e = angle * D
    b = GAIN * (D * D + e * e - RS * RS) ** 3
    speed = (-b - v * 2 * np.sqrt(2) * np.hypot(D, e)) / (4 * D)
    p = dict(x_min=-X_MAX, x_max=X_MAX, y_min=-6.0, y_max=6.0, barrier_gain=GAIN,
             safety_radius=RS, boundary_gain_factor=speed / (X_MAX - RS / 2 - D / 2) ** 3 / GAIN)
    k = np.arange(6)
    px, py, ux, uy = np.zeros((4, E, 8))
    px[:, 0], px[:, 1], py[:, 0], py[:, 1] = D / 2, -D / 2, e / 2, -e / 2
    px[:, 2:] = np.where(k % 2, 0.1, -0.1) + rng.uniform(-0.01, 0.01, (E, 6))
    py[:, 2:] = 1.0 + 0.2 * (k // 2) + rng.uniform(-0.01, 0.01, (E, 6))
    ux[:, 0], ux[:, 1] = 0.1, -0.1
    dx = px[:, 2:].mean(1, keepdims=True) - px[:, 2:]
    dy = py[:, 2:].mean(1, keepdims=True) - py[:, 2:]
    size = (1e-3 if tiny else 0.2) / np.hypot(dx, dy)
    ux[:, 2:], uy[:, 2:] = size * dx, size * dy
    return p, (px, py, ux, uy), b


# kind, v_max, angle, share of the speed limit that the pair moves at
@pytest.mark.parametrize("kind,v_max,angle,share", [
    ("f32", 0.2, 2e-5, 0.7), ("f32", 0.2, 1e-4, 0.3),
    ("f32", 50.0, 2e-6, 0.3), ("f32", 50.0, 5e-6, 0.7), ("f32", 50.0, 2e-5, 0.3),
    ("f64", 0.2, 2e-11, 0.7), ("f64", 0.2, 1e-10, 0.3),
    ("f64", 50.0, 5e-11, 0.7), ("f64", 50.0, 1e-9, 0.3), ("f64", 50.0, 1e-9, 0.7)])
def test_row_left_a_sliver_by_the_bounds(orc, kind, v_max, angle, share):
    import torch

    R, ctx = ctx_and_lib()
    tdt, ndt = (torch.float32, np.float32) if kind == "f32" else (torch.float64, np.float64)
    E, n = 64, 8
    v = share * np.sqrt(2) * v_max * angle
    kw, arrs, b = _packs(1, E, angle, v, v_max > 1)
    arrs = [a.astype(ndt) for a in arrs]
    p = R.params(dtype=R.RS_F64 if kind == "f64" else R.RS_F32, v_max=v_max, **kw)
    banner(f"thin row {kind} v_max {v_max} angle {angle}")
    ux, uy = (torch.zeros(E * n, dtype=tdt, device="cuda") for _ in range(2))
    status = torch.full((E,), 255, dtype=torch.uint8, device="cuda")
    qs = torch.zeros((E, R.QPS_COUNT), dtype=torch.int32, device="cuda")
    R.barrier_certificate(ctx, p, E, n, *(dev(a.ravel(), tdt) for a in arrs), ux, uy,
                          infeasible=status, qp_stats=qs)
    torch.cuda.synchronize()
    got = np.stack([host(t).reshape(E, n).astype(np.float64) for t in (ux, uy)])
    assert host(qs)[:, R.QPS_GENERAL].sum() == E
    assert (host(status) == 0).all()
    tol = 1e-4 if kind == "f32" else 1e-9
    # the pair's motion is the row's violation over the angle: the violation's
    # rounding (some 16 units of b over the row's norm, 2 sqrt(2) D) scaled alike
    dv = 16 * np.finfo(ndt).eps / 2 * abs(b) / (2 * np.sqrt(2) * D)
    pair_tol = tol + 4 * share * v_max * dv / v
    po = orc.Params(v_max=v_max, **kw)
    for e in range(8):
        ref = orc.barrier_certificate(po, *[a[e].astype(np.float64) for a in arrs])
        assert ref[3] == 0
        err = np.abs(got[:, e] - np.stack(ref[:2]))
        assert err[:, 2:].max() <= tol
        assert err[:, :2].max() <= pair_tol
