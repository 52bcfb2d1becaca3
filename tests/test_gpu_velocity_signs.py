"""The sign parts of the velocity gradient in the frequency advection (double, whole zones per wave):
a component below 0 has no part that is 0 or above.  In a medium that is compressed along every
component of the gradient each intergroup flux takes the lower group alone, so a group above whose
lower neighbours are empty sends nothing down: the lower groups stay exactly 0 (with no emission),
as in the oracle.  Group counts on both sides of the rule that shares the gradient among a zone's
lanes, Cartesian and spherical.  The other bounds are those of every parity case in FP64."""
import numpy as np
import pytest
import torch

from oracle import m1_oracle as orc
from paper_1806_07390_amd import workloads as wl
from tests.parity_util import TOL_FP64, problem_of, rel_l1, to_dev, to_host

pytestmark = pytest.mark.gpu

CASES = [("cart2d", g) for g in (3, 4, 22)] + [("cart3d", g) for g in (3, 4, 8, 9, 12)] \
    + [("sph2d", g) for g in (3, 6)] + [("sph3d", g) for g in (3, 8, 9, 12)]


def workload(kind, G, seed):
    rng = np.random.default_rng(seed)
    if kind == "cart2d":
        w = wl.blobs2d(n=24, G=G)
    elif kind == "cart3d":
        w = wl.core3d(n=12, G=G)
    else:
        w = wl.sphere3d(nr=24, nth=8, nph=1 if kind == "sph2d" else 8, G=G, ndim=int(kind[3]))
        w.inflow = np.zeros_like(w.inflow)
    s = (w.n[2], w.n[1], w.n[0], G)
    w.E = np.exp(rng.normal(0.0, 0.5, s))
    w.E[..., :2] = 0.0
    d = rng.normal(size=(w.ndim,) + s)
    d /= np.linalg.norm(d, axis=0)
    w.F = [np.ascontiguousarray(0.5 * rng.random(s) * w.c * w.E * d[k]) for k in range(w.ndim)]
    w.kappa, w.sigma, w.B = 0.3 * rng.random(s), 0.3 * rng.random(s), np.zeros(s)
    # on the faces of each direction every component falls along it, by another amount in every zone;
    # steeply enough that on spherical grids the connection's part changes no sign
    sph = w.coord != wl.CARTESIAN
    vf = []
    for k in range(w.ndim):
        fs = list(s[:3])
        fs[2 - k] += 1
        dx = (w.hi[k] - w.lo[k]) / w.n[k]
        v = np.empty((w.ndim,) + tuple(fs))
        for i in range(w.ndim):
            slope = 2e-6 * (1.0 if i == k else 20.0) if sph else 0.05
            fall = slope * dx * (0.8 + 0.4 * rng.random(s[:3]))
            v[i] = np.concatenate([np.zeros_like(np.take(fall, [0], 2 - k)), -np.cumsum(fall, 2 - k)], 2 - k)
            if sph and i == k:
                v[i] += -3e-5 if k == 0 else 0.5 * slope * (w.hi[k] - w.lo[k])
        vf.append(np.ascontiguousarray(v))
    return w, vf


@pytest.mark.parametrize("kind,G", CASES)
def test_sign_parts(kind, G):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1806_07390_amd import m1
    w, vf = workload(kind, G, 3 + G)
    p = problem_of(w)
    nu = np.concatenate([[0.0], np.geomspace(0.5, 20.0, G)])
    ctx = m1.Context(m1.Config.from_workload(w, precision=m1.FP64))
    ctx.set_group_edges(nu)
    dt = ctx.max_dt(0.2)
    Er, Fr, _ = orc.run_v(p, w.E, w.F, w.kappa, w.sigma, w.B, vf, nu, dt, 1, inflow=w.inflow)
    neg = np.all(orc.vel_grad(p, vf)[0][..., :w.ndim, :w.ndim] < 0, axis=(-1, -2))
    assert neg.all() and np.all(Er[..., :2] == 0)
    d = lambda a: to_dev(np.ascontiguousarray(a), torch.float64)
    infl = None if w.inflow is None else d(w.inflow)
    E, F = ctx.step_velocity(d(w.E), [d(f) for f in w.F], d(w.kappa), d(w.sigma), d(w.B), [d(v) for v in vf], dt,
                             inflow=infl)
    torch.cuda.synchronize()
    E, F = to_host(E), [to_host(f) for f in F]
    assert np.all(E[Er == 0] == 0)
    for a, b in zip(F, Fr):
        assert np.all(a[b == 0] == 0)
    eE, eF = rel_l1(E, F, Er, Fr, w.c)
    assert eE <= TOL_FP64 and eF <= TOL_FP64
