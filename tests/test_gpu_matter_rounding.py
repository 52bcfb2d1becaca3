"""Rounding of the matter kernels' results: emission in the Wien tail to what a correctly rounded
nu/T allows, and an infinitely opaque scatterer.

Bound of the emission of the top group (a, inf), which is a T^4 times one sum of positive terms
proportional to e^(-x), x = a/T: rounding x once changes e^(-x) by x 2^-53; the exponential, the
polynomial, T^4 and the products add at most 16 roundings of 2^-53."""
import numpy as np
import pytest
import torch

from tests.parity_util import to_dev, to_host

pytestmark = pytest.mark.gpu


def _ctx(m1, G, n, edges, nu_c):
    ctx = m1.Context(m1.Config(ndim=2, n=n, G=G))
    ctx.set_matter_model(edges, nu_c, np.ones(G), a_rad=1.0, tol=1e-6, max_newton=30)
    return ctx


@pytest.mark.parametrize("G", [2, 5, 16, 40])
def test_wien_tail(G):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1806_07390_amd import m1
    edges = np.concatenate([np.linspace(0.0, 30.0, G), [np.inf]])
    nu_c = np.concatenate([0.5 * (edges[:-2] + edges[1:-1]), [60.0]])
    ctx = _ctx(m1, G, (64, 32), edges, nu_c)
    rng = np.random.default_rng(G)
    T = 30.0 / np.exp(rng.uniform(np.log(5.0), np.log(650.0), (1, 32, 64)))
    d = lambda a: to_dev(np.ascontiguousarray(a), torch.float64)
    one = np.ones_like(T)
    _, B = ctx.matter_coeffs(d(one), d(one), d(T))
    L = np.longdouble
    Tl = T.astype(L)
    x = L(30.0) / Tl
    tail = np.zeros_like(x)
    for n in range(1, 40):
        n_ = L(n)
        tail += np.exp(-n_ * x) * (x ** 3 / n_ + 3 * x ** 2 / n_ ** 2 + 6 * x / n_ ** 3 + 6 / n_ ** 4)
    pi = L("3.14159265358979323846264338327950288")
    ref = Tl ** 4 * 15 / pi ** 4 * tail
    err = np.abs(to_host(B)[..., -1].astype(L) - ref) / ref
    assert np.all(err <= (x + 16) * L(2) ** -53)


@pytest.mark.parametrize("prec", [0, 1])
def test_infinite_scattering(prec):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1806_07390_amd import m1
    G, n = 5, (13, 7)
    edges = np.geomspace(0.2, 20.0, G + 1)
    ctx = m1.Context(m1.Config(ndim=2, n=n, G=G, precision=prec))
    ctx.set_matter_model(edges, np.sqrt(edges[1:] * edges[:-1]), np.ones(G), a_rad=1.0, tol=1e-6, max_newton=30)
    rng = np.random.default_rng(3)
    E = torch.from_numpy(rng.uniform(0.1, 1.0, ctx.shape)).cuda().to(ctx.dtype)
    F = [0.3 * E, -0.2 * E]
    sigma = torch.rand_like(E)
    sigma[:, ::2] = float("inf")
    zone = lambda: torch.from_numpy(rng.uniform(0.5, 2.0, ctx.shape[:3])).cuda()
    ctx.matter_source(E, F, sigma, zone(), zone(), zone(), 0.1)
    torch.cuda.synchronize()
    for f in F:
        assert torch.all(f[:, ::2] == 0) and torch.all(f[:, 1::2].abs() > 0)
    assert torch.isfinite(E).all()
