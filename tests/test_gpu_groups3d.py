"""GPU parity of the 3-D kernel where its rows hold something else than four groups of one x tile:
one and two groups (rows of four and two x tiles), and group counts that leave rows idle; grids
with a ragged last tile in every direction, Cartesian (reflecting and periodic) and spherical, FP64
and MIXED, with the diagnostics, and Step 1 of the velocity step on the same rows.

Bounds: the same as every parity case of the step (parity_util): 1e-12 relative L1 in FP64 and the
MIXED per-step bound; dE_matter is a sum over groups of differences E^{n+1} - E^-, each rounded at
the size of E, so it is held to the bound times the largest group sum of E."""
import numpy as np
import pytest
import torch

from oracle import m1_oracle as orc
from paper_1806_07390_amd import workloads as wl
from tests.parity_util import TOL_FP64, TOL_MIXED_STEP, problem_of, rel_l1, to_dev, to_host

pytestmark = pytest.mark.gpu


def _workload(grid, G, seed, big=False):
    rng = np.random.default_rng(seed)
    if grid == "sphere":
        n = (131, 34, 62) if big else (33, 10, 12)
        w = wl.sphere3d(nr=n[0], nth=n[1], nph=n[2], G=G)
        w.E = w.E * (1.0 + rng.random(w.E.shape)) + 1e-3 * rng.random(w.E.shape)
    else:
        nx, ny, nz = (53, 51, 50) if big else (19, 9, 17)
        w = wl.core3d(n=nx, G=max(G, 2), seed=seed)
        cut = lambda a: np.ascontiguousarray(a[:nz, :ny, :, :G])
        w.E, w.kappa, w.sigma, w.B = cut(w.E), cut(w.kappa), cut(w.sigma), cut(w.B)
        w.F = [0.4 * w.E * rng.uniform(-1, 1, w.E.shape) for _ in range(3)]
        w.n, w.G = (nx, ny, nz), G
        bc = wl.BC_REFLECT if grid == "reflect" else wl.BC_PERIODIC
        w.bc_lo = w.bc_hi = (bc,) * 3
    return w


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("G", [1, 2, 3, 5, 6, 7])
@pytest.mark.parametrize("grid", ["reflect", "periodic", "sphere"])
def test_step_rows(grid, G, prec):
    from paper_1806_07390_amd import m1
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    w = _workload(grid, G, 3 * G)
    if prec:
        r32 = lambda a: np.asarray(a, dtype=np.float32).astype(np.float64)
        w.E, w.F, w.kappa, w.sigma, w.B = r32(w.E), [r32(f) for f in w.F], r32(w.kappa), r32(w.sigma), r32(w.B)
    ctx = m1.Context(m1.Config.from_workload(w, precision=prec))
    dt = ctx.max_dt(0.4)
    d = lambda a: to_dev(np.ascontiguousarray(a), ctx.dtype)
    infl = None if w.inflow is None else to_dev(w.inflow, torch.float64)
    dg = ctx.new_diag()
    E, F = ctx.step(d(w.E), [d(f) for f in w.F], d(w.kappa), d(w.sigma), d(w.B), dt, inflow=infl, diag=dg)
    torch.cuda.synchronize()
    Er, Fr, diag, dEm = orc.run(problem_of(w), w.E, w.F, w.kappa, w.sigma, w.B, dt, 1, inflow=w.inflow,
                                want_dEm=True)
    eE, eF = rel_l1(to_host(E), [to_host(f) for f in F], Er, Fr, w.c)
    tol = TOL_MIXED_STEP if prec else TOL_FP64
    assert eE <= tol and eF <= tol
    assert np.abs(dg["dE_matter"].cpu().numpy() - dEm.ravel()).max() <= tol * w.G * np.abs(Er).max()
    assert abs(dg["energy_total"].item() - diag["energy_total"]) <= tol * abs(diag["energy_total"])
    assert int(dg["n_nonpositive"].item()) == diag["n_nonpositive"]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("G", [1, 2, 3])
@pytest.mark.parametrize("grid", ["reflect", "sphere"])
def test_velocity_rows(grid, G, prec):
    from paper_1806_07390_amd import m1
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    w = _workload(grid, G, 5 * G + 1, big=True)
    vf = wl.face_velocity(w, amp=0.1, seed=G)
    nu = wl.velocity_edges(G) if G > 1 else np.array([1.0, 2.0])
    ctx = m1.Context(m1.Config.from_workload(w, precision=prec))
    ctx.set_group_edges(nu)
    dt = ctx.max_dt(0.3)
    d = lambda a: to_dev(np.ascontiguousarray(a), ctx.dtype)
    infl = None if w.inflow is None else to_dev(w.inflow, torch.float64)
    E, F = ctx.step_velocity(d(w.E), [d(f) for f in w.F], d(w.kappa), d(w.sigma), d(w.B), [d(v) for v in vf], dt,
                             inflow=infl)
    torch.cuda.synchronize()
    Er, Fr, _ = orc.run_v(problem_of(w), w.E, w.F, w.kappa, w.sigma, w.B, vf, nu, dt, 1, inflow=w.inflow)
    eE, eF = rel_l1(to_host(E), [to_host(f) for f in F], Er, Fr, w.c)
    tol = TOL_MIXED_STEP if prec else TOL_FP64
    assert eE <= tol and eF <= tol
