"""GPU test of the certificate in other units of length: a problem whose arena,
radius, speeds and gains are scaled together is the same problem, so dense packs
that need the general solver are solved (status 0, nothing capped) and their
commands, scaled back, are the FP64 oracle's minimiser to the tolerances of the
default units (1e-4 m/s in FP32, 1e-9 in FP64)."""
import numpy as np
import pytest

from tests.gpu_util import banner, ctx_and_lib, dev, host
from tests.test_gpu_qp_general import _packs

pytestmark = pytest.mark.gpu

LENGTHS = ("x_min", "x_max", "y_min", "y_max", "proj_dist", "safety_radius", "v_max",
           "action_speed", "waypoint_step", "goal_radius", "reset_margin", "min_sep", "grid",
           "wheel_radius", "base_length", "prey_speed", "tag_radius")


@pytest.mark.parametrize("unit", [1, 30, 1000])
@pytest.mark.parametrize("kind", ["f32", "f64"])
@pytest.mark.parametrize("n", [5, 8, 16])
def test_dense_packs_in_other_units(orc, n, kind, unit):
    import torch

    R, ctx = ctx_and_lib()
    tdt, ndt = (torch.float32, np.float32) if kind == "f32" else (torch.float64, np.float64)
    p = R.params(dtype=R.RS_F64 if kind == "f64" else R.RS_F32)
    for f in LENGTHS:
        setattr(p, f, getattr(p, f) * unit)
    p.barrier_gain /= unit ** 4           # b = gamma h^3 is an area per time
    p.boundary_gain_factor *= unit ** 2   # the wall gain times a length cubed, a speed
    E = 1100  # the first envs against the oracle, all of them for their status
    arrs = [(a * unit).astype(ndt) for a in _packs(60 + n, E, n)]
    banner(f"dense packs n={n} {kind} unit {unit}")
    ux, uy = (torch.zeros(E * n, dtype=tdt, device="cuda") for _ in range(2))
    status = torch.full((E,), 255, dtype=torch.uint8, device="cuda")
    qs = torch.zeros((E, R.QPS_COUNT), dtype=torch.int32, device="cuda")
    R.barrier_certificate(ctx, p, E, n, *(dev(a.ravel(), tdt) for a in arrs), ux, uy,
                          infeasible=status, qp_stats=qs)
    torch.cuda.synchronize()
    gux, guy = (host(t).reshape(E, n).astype(np.float64) / unit for t in (ux, uy))
    st, qs = host(status), host(qs)
    if n >= 8:
        assert qs[:, R.QPS_GENERAL].sum() > 0
    assert (st != 2).all() and (qs[:, R.QPS_CAPPED] == 0).all()
    tol = 1e-4 if kind == "f32" else 1e-9
    po = orc.Params()
    for e in range(40):
        ref = orc.barrier_certificate(po, *[v[e].astype(np.float64) / unit for v in arrs])
        assert bool(ref[3]) == (st[e] == 1)
        assert max(np.abs(gux[e] - ref[0]).max(), np.abs(guy[e] - ref[1]).max()) <= tol
