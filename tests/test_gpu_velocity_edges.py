"""The closed ends of the frequency range in the velocity step (double, whole zones per wave): with
the lowest edge above 0, no energy crosses the lower edge of a zone's first group or the upper edge
of its last one, whatever the zone before or after it in memory holds.  Rows whose two ends lie next
to each other in memory hold radiation at one end and nothing (whole zones, or the groups next to
a closed edge) at the other, with no emission.

Where the oracle holds exactly 0 the step has to hold exactly 0.  The other bounds are those of
every parity case of the step in FP64 (1e-12 relative L1); with whole zones empty the counts are
equal and max_f is held to the same bound (with single groups empty the frequency fluxes into them
leave energies that cancel to 1e-16 of their terms, whose sign and f the bound does not fix)."""
import numpy as np
import pytest
import torch

from oracle import m1_oracle as orc
from paper_1806_07390_amd import workloads as wl
from tests.parity_util import TOL_FP64, problem_of, rel_l1, to_dev, to_host

pytestmark = pytest.mark.gpu

NX = 60
CASES = [("cart2d", g) for g in (1, 2, 3, 5, 16, 22, 64)] + [("cart3d", g) for g in (1, 4, 8, 9, 12)] \
    + [("sph2d", g) for g in (1, 6)] + [("sph3d", g) for g in (2, 9, 12)]


def workload(kind, G, empty, seed):
    """empty: "zones" (the left third of every row), "low" / "high" (the two groups next to the
    closed lower edge at the left / upper edge at the right end); the middle of a row is empty."""
    rng = np.random.default_rng(seed)
    if kind == "cart2d":
        w = wl.blobs2d(n=NX, G=G)
        w.n = (NX, 6, 1)
    elif kind == "cart3d":
        w = wl.core3d(n=NX, G=max(G, 2))
        w.n, w.G = (NX, 4, 4), G
    else:
        w = wl.sphere3d(nr=NX, nth=6, nph=1 if kind == "sph2d" else 4, G=G, ndim=int(kind[3]))
        w.inflow = np.zeros_like(w.inflow)
    s = (w.n[2], w.n[1], w.n[0], G)
    w.E = np.exp(rng.normal(0.0, 0.5, s))
    w.E[:, :, 16:NX - 16] = 0.0
    if empty == "zones":
        w.E[:, :, :16] = 0.0
    elif empty == "low":
        w.E[:, :, :16, :2] = 0.0
    else:
        w.E[:, :, NX - 16:, G - 2:] = 0.0
    d = rng.normal(size=(w.ndim,) + s)
    d /= np.linalg.norm(d, axis=0)
    w.F = [np.ascontiguousarray(0.5 * rng.random(s) * w.c * w.E * d[k]) for k in range(w.ndim)]
    w.kappa, w.sigma, w.B = 0.3 * rng.random(s), 0.3 * rng.random(s), np.zeros(s)
    return w


@pytest.mark.parametrize("steps", [1, 2, 10])
@pytest.mark.parametrize("empty", ["zones", "low", "high"])
@pytest.mark.parametrize("kind,G", CASES)
def test_closed_edges(kind, G, empty, steps):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    if G <= 2 and empty != "zones":
        pytest.skip("no group is left")
    from paper_1806_07390_amd import m1
    w = workload(kind, G, empty, 7 + G)
    vf = wl.face_velocity(w, amp=0.1, seed=G)
    nu = np.geomspace(0.5, 20.0, G + 1)
    ctx = m1.Context(m1.Config.from_workload(w, precision=m1.FP64))
    ctx.set_group_edges(nu)
    dt = ctx.max_dt(0.3)
    d = lambda a: to_dev(np.ascontiguousarray(a), torch.float64)
    infl = None if w.inflow is None else d(w.inflow)
    dg = ctx.new_diag()
    U = (d(w.E), [d(f) for f in w.F])
    k, s, B, v = d(w.kappa), d(w.sigma), d(w.B), [d(x) for x in vf]
    for _ in range(steps):
        U = ctx.step_velocity(U[0], U[1], k, s, B, v, dt, inflow=infl, diag=dg)
    torch.cuda.synchronize()
    Er, Fr, diag = orc.run_v(problem_of(w), w.E, w.F, w.kappa, w.sigma, w.B, vf, nu, dt, steps, inflow=w.inflow)
    assert (Er == 0).any()
    E, F = to_host(U[0]), [to_host(f) for f in U[1]]
    assert np.all(E[Er == 0] == 0)
    for a, b in zip(F, Fr):
        assert np.all(a[b == 0] == 0)
    eE, eF = rel_l1(E, F, Er, Fr, w.c)
    assert eE <= TOL_FP64 and eF <= TOL_FP64
    if empty != "zones":
        return
    assert int(dg["n_nonpositive"].item()) == diag["n_nonpositive"]
    assert int(dg["n_unrealizable"].item()) == diag["n_unrealizable"]
    assert abs(dg["max_f"].item() - diag["max_f"]) <= TOL_FP64 * diag["max_f"]


@pytest.mark.parametrize("kind,G", [("cart2d", 2), ("cart2d", 5), ("cart3d", 8), ("cart3d", 9)])
def test_subnormal_energies(kind, G):
    """Energies below the smallest normal number (what is left in a zone that empties) stay finite and
    follow the oracle.  An operation rounds such values by up to 2.5e-324; a few hundred of them per
    step, each at most doubled by a later one, stay below 1e-320 (the state: 1e-310)."""
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1806_07390_amd import m1
    w = workload(kind, G, "zones", 11 + G)
    rng = np.random.default_rng(G)
    w.E = 1e-310 * rng.random(w.E.shape)
    w.F = [0.5 * w.c * w.E * rng.uniform(-1, 1, w.E.shape) for _ in range(w.ndim)]
    vf = wl.face_velocity(w, amp=0.1, seed=G)
    nu = np.geomspace(0.5, 20.0, G + 1)
    ctx = m1.Context(m1.Config.from_workload(w, precision=m1.FP64))
    ctx.set_group_edges(nu)
    dt = ctx.max_dt(0.3)
    d = lambda a: to_dev(np.ascontiguousarray(a), torch.float64)
    E, F = ctx.step_velocity(d(w.E), [d(f) for f in w.F], d(w.kappa), d(w.sigma), d(w.B), [d(x) for x in vf], dt)
    torch.cuda.synchronize()
    Er, Fr, _ = orc.run_v(problem_of(w), w.E, w.F, w.kappa, w.sigma, w.B, vf, nu, dt, 1)
    assert np.isfinite(Er).all() and np.abs(to_host(E) - Er).max() <= 1e-320
    for a, b in zip(F, Fr):
        assert np.abs(to_host(a) - b).max() <= 1e-320
