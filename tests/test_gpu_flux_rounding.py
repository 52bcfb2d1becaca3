"""The energy flux between nearly equal states at rest, -(c/2) (E_R - E_L) where the zones are
transparent: the difference of two energies a few ulp apart is exact, so the flux is good to a few
ulp of itself, not of c E.  Bound: 8 operations of half an ulp (2^-53) each, 1e-15; the spherical
faces' scale factors are two more tables and reciprocals of a few ulp, 1e-14."""
import numpy as np
import pytest
import torch

from oracle import m1_oracle as orc
from paper_1806_07390_amd import workloads as wl
from tests.parity_util import problem_of, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c", [1.0, 0.7, 2.99792458e10])
@pytest.mark.parametrize("kind", ["cart1d", "cart2d", "cart3d", "sph3d"])
def test_energy_flux_of_nearly_equal_states(kind, c):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1806_07390_amd import m1
    G = 3
    if kind == "sph3d":
        w = wl.sphere3d(nr=10, nth=6, nph=4, G=G)
        w.inflow = np.concatenate([np.full((G, 1), 1.0), np.zeros((G, 3))], axis=1)
    else:
        w = {"cart1d": lambda: wl.slab1d(n=40, G=G), "cart2d": lambda: wl.blobs2d(n=14, G=G),
             "cart3d": lambda: wl.core3d(n=9, G=G)}[kind]()
    w.c = c
    s = (w.n[2], w.n[1], w.n[0], G)
    rng = np.random.default_rng(5)
    E = 1.3 + rng.integers(-9, 10, s) * 2.0 ** -52
    Z = np.zeros(s)
    F = [Z.copy() for _ in range(w.ndim)]
    p = problem_of(w)
    p.limiter = 2
    ctx = m1.Context(m1.Config.from_workload(w, precision=m1.FP64, limiter=m1.LIMITER_NONE))
    d = lambda a: to_dev(np.ascontiguousarray(a), torch.float64)
    infl = None if w.inflow is None else d(w.inflow)
    out = ctx.flux(d(E), [d(f) for f in F], d(Z), d(Z), d(Z), inflow=infl)
    torch.cuda.synchronize()
    tol = 1e-14 if kind == "sph3d" else 1e-15
    for k in range(w.ndim):
        ref = orc.flux(p, E, F, Z, Z, Z, k, inflow=w.inflow)[..., 0]
        got = to_host(out[k])[..., 0]
        assert np.count_nonzero(ref) > 0
        assert np.all(np.abs(got - ref) <= tol * np.abs(ref))
