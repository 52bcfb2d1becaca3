"""GPU parity of the matter kernels where their lane layout and Planck series change: group counts
on both sides of each lane count per zone (1 to 64 lanes), a finite and an infinite top edge (a
zone's last lane then does or does not evaluate it), temperatures that put a group edge exactly
at, just below and just above the split of the two series, and cold and hot zones (every edge on
one side of it).

Bounds: the coefficients are direct evaluations in double; an edge value carries a few ulp of a
series summing to at most twice the group's integral for groups an e-fold or less apart, and
e^(-x) a relative error of x ulp (x <= 50 here), below 1e-13 together.  The temperatures stop at
Newton steps of 1e-6, whose square is the error left (1e-9, as for the other matter cases)."""
import numpy as np
import pytest
import torch

from oracle import m1_oracle as orc
from tests.parity_util import to_dev, to_host

pytestmark = pytest.mark.gpu

SPLIT = 3.5


def _tables(G, finite_top):
    inner = np.geomspace(0.3, 12.0, G - 1) if G > 2 else np.array([3.0][:G - 1])
    edges = np.concatenate([[0.0], inner, [20.0 if finite_top else np.inf]])
    nu_c = np.where(np.isfinite(edges[1:]), 0.5 * (edges[:-1] + np.minimum(edges[1:], 1e3)), 2.0 * edges[:-1] + 1.0)
    return edges, nu_c, (nu_c / 2.821) ** -2


@pytest.mark.parametrize("finite_top", [False, True])
@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64])
def test_lanes_per_zone(G, finite_top):
    from paper_1806_07390_amd import m1
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    edges, nu_c, kg = _tables(G, finite_top)
    rng = np.random.default_rng(G)
    T = np.exp(0.4 * rng.standard_normal((1, 9, 13)))
    flat = T.reshape(-1)
    at = edges[1:-1][: 20] / SPLIT
    for k, t in enumerate(at):
        flat[3 * k:3 * k + 3] = (t, np.nextafter(t, 0.0), np.nextafter(t, 9.0))
    flat[-2:] = (0.4, 9.0)
    z = T.shape
    E = rng.uniform(0.0, 0.5, z + (G,))
    F = [0.3 * E * rng.uniform(-1, 1, z + (G,)) for _ in range(2)]
    sigma, cv, k0 = rng.uniform(0, 2, z + (G,)), np.exp(0.5 * rng.standard_normal(z)), np.exp(rng.standard_normal(z))
    mod = orc.MatterModel(edges, nu_c, kg, a_rad=1.0, c=1.0, tol=1e-6, max_newton=30)
    ctx = m1.Context(m1.Config(ndim=2, n=(13, 9), G=G))
    ctx.set_matter_model(edges, nu_c, kg, a_rad=1.0, tol=1e-6, max_newton=30)
    d = lambda a: to_dev(np.ascontiguousarray(a), torch.float64)
    kap, B = ctx.matter_coeffs(d(cv), d(k0), d(T))
    kr, Br = orc.matter_coeffs(mod, k0, T)
    assert np.abs(to_host(kap) - kr).max() <= 1e-13 * np.abs(kr).max()
    assert np.all(np.abs(to_host(B) - Br) <= 1e-13 * np.abs(Br) + 1e-15 * np.abs(Br).max())
    Er, Fr, Tr, dr, itr = orc.matter_source(mod, E, F, sigma, cv, k0, T, 0.2)
    Eg, Fg, Tg = d(E), [d(f) for f in F], d(T)
    dg = torch.zeros(ctx.nzones, dtype=torch.float64, device="cuda")
    ctx.matter_source(Eg, Fg, d(sigma), d(cv), d(k0), Tg, 0.2, dE_matter=dg)
    torch.cuda.synchronize()
    assert np.allclose(to_host(Tg), Tr, rtol=1e-9, atol=0)
    assert np.abs(to_host(Eg) - Er).max() <= 1e-9 * np.abs(Er).max()
    for a, b in zip(Fg, Fr):
        assert np.abs(to_host(a) - b).max() <= 1e-9 * np.abs(Er).max()
    assert np.abs(to_host(dg) - dr.ravel()).max() <= 1e-9 * np.abs(cv * T).max()
