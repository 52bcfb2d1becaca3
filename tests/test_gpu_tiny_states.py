"""The diagnostics of states far below any physical size: the largest f and the counts do not depend on
the scale of (E, F).  A zone's f is compared with the largest one so far by products of two
squared energies, which underflow below about 1e-81.  Every kernel that has its own reduction
of the diagnostics: 1-D and 2-D tiles, whole-zone rows (2-D, 16 groups), the 3-D plane kernel, spherical
grids, both integrators, the velocity step by wave and by block (65 groups).

The scale is a power of two above the one at which the step's own realizability checks (squares of
the state) underflow, so the scaled run repeats the roundings of the unscaled one: max_f to
1e-12, equal counts."""
import numpy as np
import pytest
import torch

from paper_1806_07390_amd import workloads as wl
from tests.parity_util import to_dev

pytestmark = pytest.mark.gpu

KINDS = ["cart1d", "cart2d-5", "cart2d-16", "cart2d-rk2", "cart3d", "sph2d", "sph3d", "vel2d", "vel2d-65"]


def workload(kind):
    rng = np.random.default_rng(len(kind))
    if kind == "cart1d":
        w = wl.slab1d(n=200, G=4)
    elif kind == "cart3d":
        w = wl.core3d(n=17, G=4)
    elif kind.startswith("sph"):
        w = wl.sphere3d(nr=20, nth=8, nph=1 if kind == "sph2d" else 8, G=4, ndim=int(kind[3]))
        w.inflow = np.zeros_like(w.inflow)
    else:
        w = wl.blobs2d(n=40, G={"cart2d-16": 16, "vel2d-65": 65}.get(kind, 5))
    s = (w.n[2], w.n[1], w.n[0], w.G)
    w.E = np.exp(rng.normal(0.0, 0.4, s))
    d = rng.normal(size=(w.ndim,) + s)
    d /= np.linalg.norm(d, axis=0)
    f = rng.uniform(0.1, 0.95, s)
    w.F = [np.ascontiguousarray(f * w.c * w.E * d[k]) for k in range(w.ndim)]
    if w.coord != wl.CARTESIAN:
        # covariant components: F_k = h_k F^_k with h_r = r at the zone centres (theta, phi left 0)
        r = np.exp(w.lo[0] + (w.hi[0] - w.lo[0]) * (np.arange(w.n[0]) + 0.5) / w.n[0])[None, None, :, None]
        w.F = [0.9 * f * w.c * w.E * r] + [np.zeros(s) for _ in range(w.ndim - 1)]
    w.E[rng.random(s) < 0.02] *= -1.0
    w.kappa, w.sigma, w.B = 0.2 * rng.random(s), 0.2 * rng.random(s), np.zeros(s)
    return w


@pytest.mark.parametrize("k", [-270, -330, -450])
@pytest.mark.parametrize("kind", KINDS)
def test_diagnostics_of_tiny_states(kind, k):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1806_07390_amd import m1
    w = workload(kind)
    ctx = m1.Context(m1.Config.from_workload(w, precision=m1.FP64,
                                             integrator=m1.SSPRK2 if kind.endswith("rk2") else m1.EULER))
    d = lambda a: to_dev(np.ascontiguousarray(a), torch.float64)
    kap, sig, B = d(w.kappa), d(w.sigma), d(w.B)
    infl = None if w.inflow is None else d(w.inflow)
    dt = ctx.max_dt(0.05)
    vel = kind.startswith("vel")
    if vel:
        ctx.set_group_edges(np.geomspace(0.5, 20.0, w.G + 1))
        vf = [d(v) for v in wl.face_velocity(w, amp=0.02, seed=1)]
    out = []
    for sc in (1.0, 2.0 ** k):
        dg = ctx.new_diag()
        E, F = d(w.E * sc), [d(f * sc) for f in w.F]
        if vel:
            ctx.step_velocity(E, F, kap, sig, B, vf, dt, inflow=infl, diag=dg)
        else:
            ctx.step(E, F, kap, sig, B, dt, inflow=infl, diag=dg)
        torch.cuda.synchronize()
        out.append((dg["max_f"].item(), dg["n_unrealizable"].item(), dg["n_nonpositive"].item()))
    assert out[0][0] > 0.5
    assert abs(out[1][0] - out[0][0]) <= 1e-12 * out[0][0]
    assert out[1][1:] == out[0][1:]
