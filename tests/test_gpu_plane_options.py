"""GPU parity of the 3-D plane kernel's rows of one and two groups (four and two x tiles) and of rows
left idle, in double, with the options that run another instantiation or a second Runge-Kutta
stage: SSP-RK2 with minmod and with PPM, MC with the M1 wavespeeds; Cartesian and spherical, with every
diagnostic.  The tiling is set, so that the plane kernel runs whichever kernel these grids would
take.  A second test gives the velocity step's frequency kernel unrealizable states on spherical
grids (|F^| up to 1.2 c E, in every direction).

Bounds: those of every parity case of the step in FP64 (1e-12 relative L1); dE_matter is a sum over
groups of differences each rounded at the size of E: the bound times the group count times the
largest |E|.  max_f = |F^|/(c E) of one zone: its relative error is that of the energy, whose error is
measured against energies max_f times larger where the step has drained the zone: the bound times
max(1, max_f)."""
import numpy as np
import pytest
import torch

from oracle import m1_oracle as orc
from paper_1806_07390_amd import workloads as wl
from tests.parity_util import TOL_FP64, problem_of, rel_l1, to_dev, to_host

pytestmark = pytest.mark.gpu

OPTS = {"rk2": dict(integrator=1), "rk2-ppm": dict(integrator=1, limiter=3), "mc-m1": dict(limiter=1, wavespeed=1)}


def _state(w, rng, fmax):
    """Energies over two decades and fluxes of every direction, |F^| up to fmax c E."""
    s = (w.n[2], w.n[1], w.n[0], w.G)
    w.E = np.exp(rng.normal(0.0, 0.8, s))
    d = rng.normal(size=(w.ndim,) + s)
    d /= np.linalg.norm(d, axis=0)
    f = fmax * rng.random(s)
    h = orc.geometry(problem_of(w))["hcell"] if w.coord != wl.CARTESIAN else np.ones(s[:3] + (3,))
    w.F = [np.ascontiguousarray(h[..., k, None] * f * w.c * w.E * d[k]) for k in range(w.ndim)]


def _check(w, dg, E, F, Er, Fr, diag, dEm):
    eE, eF = rel_l1(to_host(E), [to_host(f) for f in F], Er, Fr, w.c)
    assert eE <= TOL_FP64 and eF <= TOL_FP64
    assert np.abs(dg["dE_matter"].cpu().numpy() - dEm.ravel()).max() <= TOL_FP64 * w.G * np.abs(Er).max()
    assert abs(dg["energy_total"].item() - diag["energy_total"]) <= TOL_FP64 * abs(diag["energy_total"])
    assert abs(dg["max_f"].item() - diag["max_f"]) <= TOL_FP64 * diag["max_f"] * max(1.0, diag["max_f"])
    assert int(dg["n_nonpositive"].item()) == diag["n_nonpositive"]
    assert int(dg["n_unrealizable"].item()) == diag["n_unrealizable"]


@pytest.mark.parametrize("opts", sorted(OPTS))
@pytest.mark.parametrize("G", [1, 2, 3, 5])
@pytest.mark.parametrize("grid", ["reflect", "periodic", "sphere"])
def test_options(grid, G, opts, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1806_07390_amd import m1
    rng = np.random.default_rng(11 * G)
    if grid == "sphere":
        w = wl.sphere3d(nr=33, nth=10, nph=12, G=G)
    else:
        w = wl.core3d(n=19, G=max(G, 2), seed=G)
        w.n, w.G = (19, 9, 17), G
        w.kappa, w.sigma, w.B = (np.ascontiguousarray(a[:17, :9, :, :G]) for a in (w.kappa, w.sigma, w.B))
        w.bc_lo = w.bc_hi = (wl.BC_REFLECT if grid == "reflect" else wl.BC_PERIODIC,) * 3
    _state(w, rng, 1.1)
    monkeypatch.setenv("FORNAX_M1_C3", "8,8")
    ctx = m1.Context(m1.Config.from_workload(w, precision=m1.FP64, **OPTS[opts]))
    dt = ctx.max_dt(0.3)
    d = lambda a: to_dev(np.ascontiguousarray(a), torch.float64)
    infl = None if w.inflow is None else d(w.inflow)
    dg = ctx.new_diag()
    E, F = ctx.step(d(w.E), [d(f) for f in w.F], d(w.kappa), d(w.sigma), d(w.B), dt, inflow=infl, diag=dg)
    torch.cuda.synchronize()
    _check(w, dg, E, F, *orc.run(problem_of(w, **OPTS[opts]), w.E, w.F, w.kappa, w.sigma, w.B, dt, 1, inflow=w.inflow,
                                 want_dEm=True))


@pytest.mark.parametrize("ndim,G", [(2, 3), (2, 4), (2, 33), (3, 2), (3, 8), (3, 9), (3, 33)])
def test_velocity_unrealizable_on_spherical_grids(ndim, G):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1806_07390_amd import m1
    w = wl.sphere3d(nr=14, nth=6, nph=1 if ndim == 2 else 6, G=G, ndim=ndim)
    _state(w, np.random.default_rng(G), 1.2)
    vf = wl.face_velocity(w, amp=0.15, seed=G)
    nu = np.geomspace(0.5, 20.0, G + 1)
    ctx = m1.Context(m1.Config.from_workload(w, precision=m1.FP64))
    ctx.set_group_edges(nu)
    dt = ctx.max_dt(0.3)
    d = lambda a: to_dev(np.ascontiguousarray(a), torch.float64)
    dg = ctx.new_diag()
    E, F = ctx.step_velocity(d(w.E), [d(f) for f in w.F], d(w.kappa), d(w.sigma), d(w.B), [d(v) for v in vf], dt,
                             inflow=d(w.inflow), diag=dg)
    torch.cuda.synchronize()
    _check(w, dg, E, F, *orc.run_v(problem_of(w), w.E, w.F, w.kappa, w.sigma, w.B, vf, nu, dt, 1, inflow=w.inflow,
                                   want_dEm=True))
